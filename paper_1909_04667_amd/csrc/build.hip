// Tree build for gfx950 (Sec. 3.1 of the Arepo paper: enclosing cube, a tree
// rebuilt for every force computation, monopole moments; Sec. 8: Peano-
// Hilbert ordering).
//
// Instead of inserting particles one by one, the tree is derived from the
// sorted 63-bit keys: a node is a key prefix shared by at least two particles,
// which is exactly the tree sequential insertion produces.  Every particle
// starts the nodes whose prefix level lies between its common-prefix depths
// with its left and right neighbours, so one scan over per-particle counts
// gives the depth-first position of every entry; a subtree ends (its skip
// pointer) at the first later entry that is not deeper.
#include "tpm_internal.h"

#include <algorithm>
#include <cstring>
#include <vector>

namespace tpm {
namespace {

constexpr int kBlock = 256;

// ---- root cube -------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_bbox_partial(const double *__restrict__ x,
                                                         const double *__restrict__ y,
                                                         const double *__restrict__ z,
                                                         int64_t n, double *__restrict__ part) {
    __shared__ double s[6][kBlock];
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    const double *c[3] = {x, y, z};
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock) {
#pragma unroll
        for (int a = 0; a < 3; a++) {
            double v = c[a][i];
            lo[a] = fmin(lo[a], v);
            hi[a] = fmax(hi[a], v);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; a++) {
        s[a][threadIdx.x] = lo[a];
        s[3 + a][threadIdx.x] = hi[a];
    }
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
#pragma unroll
            for (int a = 0; a < 3; a++) {
                s[a][threadIdx.x] = fmin(s[a][threadIdx.x], s[a][threadIdx.x + w]);
                s[3 + a][threadIdx.x] = fmax(s[3 + a][threadIdx.x], s[3 + a][threadIdx.x + w]);
            }
        }
        __syncthreads();
    }
    if (threadIdx.x < 6)
        part[blockIdx.x * 6 + threadIdx.x] = s[threadIdx.x][0];
}

// Smallest power of two >= ext (1 + 2^-20) (1 when every particle coincides);
// the corner sits below the minimum by a fraction shift of the slack.
__device__ __forceinline__ void make_frame(const double lo[3], const double hi[3], double s0,
                                           double s1, double s2, Frame &F) {
    double ext = 0.0;
    for (int a = 0; a < 3; a++) {
        double e = hi[a] - lo[a];
        ext = e > ext ? e : ext;
    }
    double L = 1.0;
    if (ext > 0.0) {
        double t = ext * (1.0 + 0x1p-20);
        int ex;
        double m = frexp(t, &ex);
        L = (m == 0.5) ? ldexp(1.0, ex - 1) : ldexp(1.0, ex);
    }
    const double shift[3] = {s0, s1, s2};
    for (int a = 0; a < 3; a++)
        F.x0[a] = lo[a] - shift[a] * (L - (hi[a] - lo[a]));
    F.L = L;
    F.S = 2097152.0 / L;
    F.box = 0.0;
    F.periodic = 0;
    F.pad = 0;
}

__global__ __launch_bounds__(kBlock) void k_frame_final(const double *__restrict__ part,
                                                        int nparts, Frame *F, double s0,
                                                        double s1, double s2) {
    // min/max of the block partials: strided over the threads, then a tree in
    // LDS (both exact, so the order does not matter)
    __shared__ double sh[6][kBlock];
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int b = threadIdx.x; b < nparts; b += kBlock)
        for (int a = 0; a < 3; a++) {
            lo[a] = fmin(lo[a], part[b * 6 + a]);
            hi[a] = fmax(hi[a], part[b * 6 + 3 + a]);
        }
    for (int a = 0; a < 3; a++) {
        sh[a][threadIdx.x] = lo[a];
        sh[3 + a][threadIdx.x] = hi[a];
    }
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w)
            for (int a = 0; a < 3; a++) {
                sh[a][threadIdx.x] = fmin(sh[a][threadIdx.x], sh[a][threadIdx.x + w]);
                sh[3 + a][threadIdx.x] = fmax(sh[3 + a][threadIdx.x], sh[3 + a][threadIdx.x + w]);
            }
        __syncthreads();
    }
    if (threadIdx.x != 0)
        return;
    for (int a = 0; a < 3; a++) {
        lo[a] = sh[a][0];
        hi[a] = sh[3 + a][0];
    }
    make_frame(lo, hi, s0, s1, s2, *F);
}

__global__ void k_set_frame(Frame h, Frame *F) { *F = h; }

// ---- keys ------------------------------------------------------------------

// Tree-frame coordinate and 21-bit cell index of one coordinate value.
__device__ __forceinline__ void to_frame(double xv, double x0, const Frame &F, double &p,
                                         uint32_t &q) {
    p = xv;
    double u = p - x0;
    if (F.periodic) {
        if (u >= F.L) {
            p = xv - F.L;
            u = p - x0;
        } else if (u < 0.0) {
            p = xv + F.L;
            u = p - x0;
        }
    }
    double f = floor(u * F.S);
    f = fmax(f, 0.0);
    f = fmin(f, 2097151.0);
    q = (uint32_t)f;
}

// Spread the low 21 bits of v to every third bit.
__device__ __forceinline__ uint64_t dilate3(uint32_t v) {
    uint64_t x = v & 0x1fffffu;
    x = (x | (x << 32)) & 0x1f00000000ffffull;
    x = (x | (x << 16)) & 0x1f0000ff0000ffull;
    x = (x | (x << 8)) & 0x100f00f00f00f00full;
    x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

// Peano-Hilbert index of a 21-bit cell (Skilling 2004, transpose form),
// branch-free: each level either inverts the low bits of axis 0 or exchanges
// them with the axis whose bit is clear; the closing Gray-code correction is
// a suffix parity computed with shifts.
__device__ __forceinline__ uint64_t hilbert_key(uint32_t a0, uint32_t a1, uint32_t a2) {
    uint32_t X0 = a0, X1 = a1, X2 = a2;
#pragma unroll
    for (int b = kBits - 1; b >= 1; --b) {
        const uint32_t P = (1u << b) - 1u;
        const uint32_t m0 = 0u - ((X0 >> b) & 1u);
        X0 ^= P & m0;
        const uint32_t m1 = 0u - ((X1 >> b) & 1u);
        const uint32_t t1 = (X0 ^ X1) & P & ~m1;
        X0 ^= (P & m1) | t1;
        X1 ^= t1;
        const uint32_t m2 = 0u - ((X2 >> b) & 1u);
        const uint32_t t2 = (X0 ^ X2) & P & ~m2;
        X0 ^= (P & m2) | t2;
        X2 ^= t2;
    }
    X1 ^= X0;
    X2 ^= X1;
    uint32_t z = X2;  // z_j = parity of bits >= j of X2
    z ^= z >> 1;
    z ^= z >> 2;
    z ^= z >> 4;
    z ^= z >> 8;
    z ^= z >> 16;
    const uint32_t t = z >> 1;
    X0 ^= t;
    X1 ^= t;
    X2 ^= t;
    return (dilate3(X0) << 2) | (dilate3(X1) << 1) | dilate3(X2);
}

// Keys, and the caller's position and mass of each particle packed into one
// 32-byte record (caller order), so that the gather into curve order reads
// one record per particle instead of four scattered values.
__global__ __launch_bounds__(kBlock) void k_keys(const double *__restrict__ x,
                                                 const double *__restrict__ y,
                                                 const double *__restrict__ z,
                                                 const double *__restrict__ mass, int64_t n,
                                                 const Frame *__restrict__ Fp,
                                                 uint64_t *__restrict__ key,
                                                 uint32_t *__restrict__ idx,
                                                 double4 *__restrict__ xyzm) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n)
        return;
    const Frame F = *Fp;
    const double xi = x[i], yi = y[i], zi = z[i];
    double p;
    uint32_t q0, q1, q2;
    to_frame(xi, F.x0[0], F, p, q0);
    to_frame(yi, F.x0[1], F, p, q1);
    to_frame(zi, F.x0[2], F, p, q2);
    key[i] = hilbert_key(q0, q1, q2);
    idx[i] = (uint32_t)i;
    xyzm[i] = make_double4(xi, yi, zi, mass ? mass[i] : 1.0 / (double)n);
}

// ---- gather into curve order -------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_gather(
    const double4 *__restrict__ xyzm, int64_t n, const Frame *__restrict__ Fp,
    const uint32_t *__restrict__ sidx, int32_t *__restrict__ perm, int32_t *__restrict__ rank,
    double *__restrict__ ps, double *__restrict__ ms, uint64_t *__restrict__ qs,
    const double *__restrict__ eps, double *__restrict__ hs, uint32_t *__restrict__ bad_eps) {
    int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (s >= n)
        return;
    const Frame F = *Fp;
    const uint32_t i = sidx[s];
    perm[s] = (int32_t)i;
    rank[i] = (int32_t)s;
    const double4 r = xyzm[i];
    double p0, p1, p2;
    uint32_t q0, q1, q2;
    to_frame(r.x, F.x0[0], F, p0, q0);
    to_frame(r.y, F.x0[1], F, p1, q1);
    to_frame(r.z, F.x0[2], F, p2, q2);
    ps[s] = p0;
    ps[n + s] = p1;
    ps[2 * n + s] = p2;
    ms[s] = r.w;
    qs[s] = ((uint64_t)q0 << 42) | ((uint64_t)q1 << 21) | (uint64_t)q2;
    if (eps) {  // individual softening: spline support 2.8 eps, in curve order
        const double e = eps[i];
        if (!(e > 0.0) || !isfinite(e))
            atomicOr(bad_eps, 1u);
        hs[s] = 2.8 * e;
    }
}

// ---- topology ----------------------------------------------------------------

// Number of leading 3-bit groups two keys share (0..21).
__device__ __forceinline__ int common_levels(uint64_t a, uint64_t b) {
    uint64_t d = a ^ b;
    if (d == 0)
        return kMaxLevel;
    int top = 63 - __clzll((long long)d);
    return (kMaxLevel - 1) - top / 3;
}

// The smallest depth shared by neighbours from this thread's particle to the
// end of its workgroup's kBlock particles (r: the depth shared with the right
// neighbour).  A node of level lev ends inside them if lev is larger.
__device__ __forceinline__ int suffix_min(int r, int *s_w) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int m = r;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_down(m, o, 64);
        m = lane + o < 64 ? min(m, t) : m;
    }
    if (lane == 0)
        s_w[w] = m;
    __syncthreads();
    for (int q = w + 1; q < kBlock / 64; q++)
        m = min(m, s_w[q]);
    __syncthreads();
    return m;
}

// Per particle: depth shared with the right neighbour, entries it starts
// (nodes at levels (dL, dR] plus itself), and per block and level the number
// of nodes its particles start that end beyond the block: hist[level * nb + block]
// (a counting sort by level, so node lists come out in particle order without
// global atomics).  The others' moments are summed where they are emitted.
__global__ __launch_bounds__(kBlock) void k_count(const uint64_t *__restrict__ key, int64_t n,
                                                  int8_t *__restrict__ dR,
                                                  uint32_t *__restrict__ cnt,
                                                  uint32_t *__restrict__ hist, uint32_t nb) {
    __shared__ uint32_t h[kLevels][kBlock / 64];
    __shared__ int s_w[kBlock / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    int r = -1, l = -1;
    if (s < n) {
        const uint64_t k = key[s];
        r = (s + 1 < n) ? common_levels(k, key[s + 1]) : -1;
        l = (s > 0) ? common_levels(key[s - 1], k) : -1;
        dR[s] = (int8_t)r;
        const int nn = r > l ? r - l : 0;
        cnt[s] = (uint32_t)nn + 1u;
    }
    const int top = min(r, suffix_min(r, s_w));
    for (int lev = 0; lev < kLevels; lev++) {
        const uint64_t m = __ballot(lev > l && lev <= top);
        if (lane == 0)
            h[lev][w] = (uint32_t)__popcll(m);
    }
    __syncthreads();
    if (threadIdx.x < kLevels) {
        uint32_t t = 0;
#pragma unroll
        for (int q = 0; q < kBlock / 64; q++)
            t += h[threadIdx.x][q];
        hist[(size_t)threadIdx.x * nb + blockIdx.x] = t;
    }
}

// What the host waits for, written to its pinned memory: the start offset of
// every level's node list (the scanned histogram's first block, 0 .. 21), the
// entries (32) and nodes (33), the frame (64) and the softening flag (128).
__global__ void k_sizes(const uint32_t *__restrict__ off, uint32_t nb,
                        const uint32_t *__restrict__ totals, const Frame *__restrict__ Fp,
                        const uint32_t *__restrict__ bad_eps, uint32_t *hpin) {
    if (threadIdx.x < kLevels)
        hpin[threadIdx.x] = off[(size_t)threadIdx.x * nb];
    if (threadIdx.x == 32 || threadIdx.x == 33)
        hpin[threadIdx.x] = totals[threadIdx.x - 32];
    if (threadIdx.x == 34)
        *(Frame *)(hpin + 64) = *Fp;
    if (threadIdx.x == 35)
        hpin[128] = *bad_eps;
}

__device__ __forceinline__ uint64_t prefix_at(uint64_t k, int lev) {
    return k >> (3 * (kMaxLevel - lev));
}

// FP32 record of an entry: exact integer centre of its cell at level lev
// (units of L 2^-22, shifted left by sh so that 32-bit differences wrap
// modulo a periodic box), level and particle flag in the freed low bits of x.
__device__ __forceinline__ void rec32_centre(Rec32 &o, const uint32_t q[3], int lev, int sh,
                                             bool part) {
    int32_t C[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const uint32_t P = q[a] >> (kBits - lev);
        C[a] = (int32_t)(((2u * P + 1u) << (kBits - lev)));
    }
    o.cx_meta = (int32_t)((uint32_t)C[0] << sh) | lev | (part ? kRecParticle : 0);
    o.cy = (int32_t)((uint32_t)C[1] << sh);
    o.cz = (int32_t)((uint32_t)C[2] << sh);
}

// Node record without its moments: the centre of the level-lev cell that holds
// the integer position q.
__device__ __forceinline__ void node_record(Rec64 &R, const uint32_t q[3], int lev,
                                            const Frame &F) {
    const double len = ldexp(F.L, -lev);
#pragma unroll
    for (int a = 0; a < 3; a++) {
        R.cen[a] = F.x0[a] + ((double)(q[a] >> (kBits - lev)) + 0.5) * len;
        R.com[a] = 0.0;
    }
    R.mass = 0.0;
    R.skip = 0u;  // set with the moments
    R.meta = (uint32_t)lev;
}

// The entries that particle s (slot) starts, from entry b on: its nodes of
// levels l + 1 .. r (the depths it shares with its left and right neighbours;
// written here, without moments, those up to level top) and itself.  FP32
// contexts (out32 set): a particle's FP32 record is written here, a node's with
// its moments.  q: the particle's integer position.
__device__ __forceinline__ void emit_particle(
    int64_t s, int64_t n, int l, int top, int r, uint32_t b, const Frame &F,
    const double *__restrict__ ps, const double *__restrict__ ms,
    const uint64_t *__restrict__ qs, Rec64 *__restrict__ rec, uint32_t *__restrict__ efirst,
    uint32_t *__restrict__ ecount, uint32_t *__restrict__ pe, const double *__restrict__ hs,
    double *__restrict__ eh, double G, Rec32 *__restrict__ out32, float *__restrict__ eh32,
    uint32_t q[3]) {
    const int nn = r > l ? r - l : 0;
    const uint32_t ep = b + (uint32_t)nn;
    const int sh = F.periodic ? kRecShiftPer : kRecShiftIso;
    const uint64_t qq = qs[s];
    q[0] = (uint32_t)(qq >> 42) & 0x1fffffu;
    q[1] = (uint32_t)(qq >> 21) & 0x1fffffu;
    q[2] = (uint32_t)qq & 0x1fffffu;
    {
        Rec64 R;
        R.com[0] = ps[s];
        R.com[1] = ps[n + s];
        R.com[2] = ps[2 * n + s];
        R.mass = ms[s];
        R.cen[0] = R.com[0];
        R.cen[1] = R.com[1];
        R.cen[2] = R.com[2];
        R.skip = ep + 1u;
        R.meta = kParticleFlag | (uint32_t)((r > l ? r : l) + 1);
        rec[ep] = R;
        efirst[ep] = (uint32_t)s;
        ecount[ep] = 1u;
        pe[s] = ep;
        if (eh)
            eh[ep] = hs[s];
        if (out32) {  // offset from the centre of its depth-21 cell
            Rec32 o;
            rec32_centre(o, q, kMaxLevel, sh, true);
            const double len = ldexp(F.L, -kMaxLevel);
            o.dx = (float)(R.com[0] - (F.x0[0] + ((double)q[0] + 0.5) * len));
            o.dy = (float)(R.com[1] - (F.x0[1] + ((double)q[1] + 0.5) * len));
            o.dz = (float)(R.com[2] - (F.x0[2] + ((double)q[2] + 0.5) * len));
            o.gm = (float)(G * R.mass);
            o.skip = R.skip;
            out32[ep] = o;
            if (eh32)
                eh32[ep] = (float)hs[s];
        }
    }
    for (int lev = l + 1; lev <= top; ++lev) {
        const uint32_t e = b + (uint32_t)(lev - l - 1);
        Rec64 R;
        node_record(R, q, lev, F);
        rec[e] = R;
        efirst[e] = (uint32_t)s;
    }
}

// Writes node e's records from its sums over the children; k: the entry
// after its subtree, cnt: its particles, q: an integer position in it.
__device__ __forceinline__ void finish_node(Rec64 *rec, uint32_t e, uint32_t k, uint32_t cnt,
                                            uint32_t lev, Rec64 R, double M, double X0, double X1,
                                            double X2, double hmax, const uint32_t q[3],
                                            uint32_t *ecount, double *eh, double G, int sh,
                                            Rec32 *out32, float *eh32) {
    const bool leaf_parent = k - e - 1u == cnt;  // no entry below but the particles themselves
    R.mass = M;
    R.com[0] = X0 / M;
    R.com[1] = X1 / M;
    R.com[2] = X2 / M;
    R.skip = k;
    R.meta |= leaf_parent ? kLeafParentFlag : 0u;
    rec[e] = R;
    ecount[e] = cnt;
    if (eh)
        eh[e] = hmax;
    if (out32) {  // exact integer centre from the node's first particle
        Rec32 o;
        rec32_centre(o, q, (int)lev, sh, false);
        o.dx = (float)(R.com[0] - R.cen[0]);
        o.dy = (float)(R.com[1] - R.cen[1]);
        o.dz = (float)(R.com[2] - R.cen[2]);
        o.gm = (float)(G * M);
        o.cx_meta |= leaf_parent ? kRecLeafParent : 0;
        o.skip = k;
        out32[e] = o;
        if (eh32)
            eh32[e] = (float)hmax;
    }
}

// Emits the entries of kBlock particles in curve order, and sums the moments of
// the nodes that end inside them (nine in ten or more): level by level, deepest
// first, a thread per particle taking the node it starts at that level, the
// children's sums, subtree ends and particle counts in LDS, so that a record is
// written once, whole.  Summed by one launch per level, every node read its
// children's records from memory again: 256^3 clustered particles, topology and
// moments 3.11 -> 1.81 ms.  Nodes that end beyond go, without moments, to the level
// lists of k_moments.  Every entry carries a depth (nodes: their level; a
// particle: the level of the cell it occupies alone, one below its deepest
// shared prefix), and the subtree of a node of level l ends at the first later
// entry of depth <= l.  kLocal: entries that LDS holds (a block's particles
// start 1.1 to 1.7 entries each in the workloads); a block with more works on
// its records in memory.
constexpr uint32_t kLocal = 640;
template <bool MIXED>
__global__ __launch_bounds__(kBlock) void k_emit(
    int64_t n, uint32_t E, const int8_t *__restrict__ dR, const uint32_t *__restrict__ base,
    const Frame *__restrict__ Fp, const double *__restrict__ ps, const double *__restrict__ ms,
    const uint64_t *__restrict__ qs, Rec64 *rec, uint32_t *efirst, uint32_t *ecount,
    uint32_t *__restrict__ pe, const uint32_t *__restrict__ loff, uint32_t nb,
    uint32_t *__restrict__ lvl_list, const double *__restrict__ hs, double *eh, double G,
    Rec32 *out32, float *eh32) {
    __shared__ uint32_t h[kLevels][kBlock / 64];
    __shared__ int s_w[kBlock / 64];
    __shared__ uint32_t s_levels;
    __shared__ double s_m[4][kLocal], s_h[MIXED ? kLocal : 1];
    __shared__ uint32_t s_skip[kLocal];
    __shared__ uint16_t s_cnt[kLocal];
    __shared__ uint8_t s_dep[kLocal];
    const int64_t s0 = (int64_t)blockIdx.x * kBlock;
    const int64_t s = s0 + threadIdx.x, s1 = s0 + kBlock < n ? s0 + kBlock : n;
    const bool live = s < n;
    const int r = live ? (int)dR[s] : -1;
    const int l = (live && s > 0) ? (int)dR[s - 1] : -1;
    const uint32_t b = live ? base[s] : 0u;
    const uint32_t e0 = base[s0], e1 = s1 < n ? base[s1] : E;  // the block's entries
    const bool lds = e1 - e0 <= kLocal;
    const int top = min(r, suffix_min(r, s_w));  // nodes of levels (l, top] end beyond
    // level lists in particle order: block offset (scanned histogram) +
    // preceding wavefronts of the block + preceding lanes of the wavefront
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    if (threadIdx.x == 0)
        s_levels = 0u;
    for (int lev = 0; lev < kLevels; lev++) {
        const uint64_t m = __ballot(lev > l && lev <= top);
        if (lane == 0)
            h[lev][w] = (uint32_t)__popcll(m);
    }
    __syncthreads();
    for (int lev = 0; lev < kLevels; lev++) {
        const bool has = lev > l && lev <= top;
        const uint64_t m = __ballot(has);
        if (has) {
            uint32_t at = loff[(size_t)lev * nb + blockIdx.x];
            for (int q = 0; q < w; q++)
                at += h[lev][q];
            lvl_list[at + (uint32_t)__popcll(m & lt)] = b + (uint32_t)(lev - l - 1);
        }
    }
    const int from = max(l, top);  // nodes of levels (from, r] are summed here
    if (live && r > from)
        atomicOr(&s_levels, (1u << (r + 1)) - (1u << (from + 1)));
    const Frame F = *Fp;
    uint32_t q[3] = {0u, 0u, 0u};
    if (live) {
        emit_particle(s, n, l, lds ? top : r, r, b, F, ps, ms, qs, rec, efirst, ecount, pe, hs,
                      eh, G, out32, eh32, q);
        if (lds) {
            for (int lev = l + 1; lev <= r; lev++)
                s_dep[b - e0 + (uint32_t)(lev - l - 1)] = (uint8_t)lev;
            const uint32_t a = b - e0 + (uint32_t)(r > l ? r - l : 0);
            s_m[0][a] = ms[s];
            s_m[1][a] = ps[s];
            s_m[2][a] = ps[n + s];
            s_m[3][a] = ps[2 * n + s];
            if (MIXED)
                s_h[a] = hs[s];
            s_skip[a] = a + 1u;
            s_cnt[a] = 1;
            s_dep[a] = (uint8_t)((r > l ? r : l) + 1);
        }
    }
    __syncthreads();
    const int sh = F.periodic ? kRecShiftPer : kRecShiftIso;
    for (uint32_t todo = s_levels; todo;) {
        const int lev = 31 - __clz((int)todo);
        todo &= ~(1u << lev);
        if (lev > from && lev <= r) {
            const uint32_t e = b + (uint32_t)(lev - l - 1);
            double M = 0.0, X0 = 0.0, X1 = 0.0, X2 = 0.0, hmax = 0.0;
            uint32_t k, cnt;
            if (lds) {
                cnt = 0u;
                for (k = e - e0 + 1u; k < e1 - e0 && s_dep[k] > lev; k = s_skip[k]) {
                    const double mk = s_m[0][k];
                    if (MIXED)
                        hmax = s_h[k] > hmax ? s_h[k] : hmax;
                    M = M + mk;
                    X0 = fma(mk, s_m[1][k], X0);
                    X1 = fma(mk, s_m[2][k], X1);
                    X2 = fma(mk, s_m[3][k], X2);
                    cnt += s_cnt[k];
                }
                k += e0;
            } else {
                for (k = e + 1u; k < e1 && (int)(rec[k].meta & 0xffu) > lev; k = rec[k].skip) {
                    const double mk = rec[k].mass;
                    if (MIXED)
                        hmax = eh[k] > hmax ? eh[k] : hmax;
                    M = M + mk;
                    X0 = fma(mk, rec[k].com[0], X0);
                    X1 = fma(mk, rec[k].com[1], X1);
                    X2 = fma(mk, rec[k].com[2], X2);
                }
                cnt = (k < e1 ? efirst[k] : (uint32_t)s1) - (uint32_t)s;
            }
            Rec64 R;
            node_record(R, q, lev, F);
            finish_node(rec, e, k, cnt, (uint32_t)lev, R, M, X0, X1, X2, hmax, q, ecount,
                        MIXED ? eh : nullptr, G, sh, out32, eh32);
            if (lds) {
                efirst[e] = (uint32_t)s;
                const uint32_t a = e - e0;
                s_m[0][a] = M;
                s_m[1][a] = X0 / M;
                s_m[2][a] = X1 / M;
                s_m[3][a] = X2 / M;
                if (MIXED)
                    s_h[a] = hmax;
                s_skip[a] = k - e0;
                s_cnt[a] = (uint16_t)cnt;
            }
        }
        __syncthreads();
    }
}

// A node of the level lists (deepest level first): walk the children through
// their skip pointers (all deeper, so already final), sum the monopole moments in
// curve order -- M = (M1 + M2) + ..., X = fma(M_k, s_k, X), s = X / M -- and
// set the node's particle count, skip pointer and leaf-parent flag.  With individual
// softening the node also takes the largest spline support of its children.
// The particle count follows from the first particles of the node and of the
// entry after its subtree (particles of a subtree are consecutive on the
// curve), so the children's counts are not read.
// FP32 contexts (out32 set): the node's FP32 record is written too (exact
// integer centre from its first particle's cell, float offset of the centre of
// mass from it, G m, skip, leaf-parent flag).
__device__ __forceinline__ void sum_node(Rec64 *rec, uint32_t e, uint32_t E, uint32_t n,
                                         const uint32_t *efirst, uint32_t *ecount, uint32_t lev,
                                         double *eh, double G, const uint64_t *qs, int sh,
                                         Rec32 *out32, float *eh32) {
    // what does not depend on the children first, so that its loads overlap
    // the walk over them
    Rec64 R = rec[e];
    const uint32_t f = efirst[e];
    const uint64_t qq = out32 ? qs[f] : 0ull;
    double M = 0.0, X0 = 0.0, X1 = 0.0, X2 = 0.0, hmax = 0.0;
    uint32_t k = e + 1;
    while (k < E && (rec[k].meta & 0xffu) > lev) {
        if (eh)
            hmax = eh[k] > hmax ? eh[k] : hmax;
        const double mk = rec[k].mass;
        M = M + mk;
        X0 = fma(mk, rec[k].com[0], X0);
        X1 = fma(mk, rec[k].com[1], X1);
        X2 = fma(mk, rec[k].com[2], X2);
        k = rec[k].skip;
    }
    const uint32_t q[3] = {(uint32_t)(qq >> 42) & 0x1fffffu, (uint32_t)(qq >> 21) & 0x1fffffu,
                           (uint32_t)qq & 0x1fffffu};
    finish_node(rec, e, k, (k < E ? efirst[k] : n) - f, lev, R, M, X0, X1, X2, hmax, q, ecount, eh,
                G, sh, out32, eh32);
}

__global__ __launch_bounds__(kBlock) void k_moments(Rec64 *rec, uint32_t E, uint32_t n,
                                                    const uint32_t *efirst, uint32_t *ecount,
                                                    const uint32_t *__restrict__ list,
                                                    uint32_t count, uint32_t lev, double *eh,
                                                    double G, const uint64_t *__restrict__ qs,
                                                    int sh, Rec32 *out32, float *eh32) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < count)
        sum_node(rec, list[i], E, n, efirst, ecount, lev, eh, G, qs, sh, out32, eh32);
}

// Consecutive levels of at most kRunNodes nodes each in one launch by one
// workgroup, a barrier between them: a launch of its own takes each level 7 us,
// however few its nodes, against 5 here (moments of 100,000 particles 125 -> 104
// us, of 50,001 78 -> 63; with 1024 nodes a level, of 2^20 157 -> 181).
constexpr int kRunNodes = 256;
struct LevelOffsets {
    uint32_t off[kLevels + 1];
};
__global__ __launch_bounds__(kRunNodes) void k_moments_run(
    Rec64 *rec, uint32_t E, uint32_t n, const uint32_t *efirst, uint32_t *ecount,
    const uint32_t *__restrict__ list, LevelOffsets lo, int deepest, int top, double *eh, double G,
    const uint64_t *__restrict__ qs, int sh, Rec32 *out32, float *eh32) {
    for (int lev = deepest; lev >= top; lev--) {
        const uint32_t i = lo.off[lev] + threadIdx.x;
        if (lo.off[lev] == lo.off[lev + 1])
            continue;
        if (i < lo.off[lev + 1])
            sum_node(rec, list[i], E, n, efirst, ecount, (uint32_t)lev, eh, G, qs, sh, out32, eh32);
        __syncthreads();
    }
}

// ---- trees of at most kSmallN particles: one workgroup ---------------------------
//
// Every pass of a small build is shorter than a launch and its gap: 35 launches
// took 0.24 ms for 4096 particles.  One workgroup takes the particles from the
// positions to the entry counts (root cube, keys, the eight digit passes of the
// sort in LDS, gather, counts and their scan), a second one, after the sizes are
// known on the host, emits the entries and sums the moments level by level.
// Same operations per particle and node as the general kernels, so the same
// tree bit for bit.  Above kSmallN the general kernels' parallel passes win.
constexpr int kSmallBlock = 1024;
constexpr int kSmallRounds = 8;
constexpr int kSmallN = kSmallBlock * kSmallRounds;
constexpr int kSmallWaves = kSmallBlock / 64;
constexpr uint32_t kSmallE = 16384;  // entries whose skip pointers fit in LDS

__device__ __forceinline__ uint32_t wave_scan(uint32_t v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(v, o, 64);
        v += lane >= o ? t : 0u;
    }
    return v;
}

// sizes: 64 words, level starts 0 .. 21, entries (32), nodes (33), also
// written to host memory with the frame (hpin + 64) and the softening flag (128).
__global__ __launch_bounds__(kSmallBlock) void k_small_front(
    const double *__restrict__ x, const double *__restrict__ y, const double *__restrict__ z,
    const double *__restrict__ mass, const double *__restrict__ eps, int n, Frame F0, double s0,
    double s1, double s2, Frame *__restrict__ Fp, uint64_t *__restrict__ key,
    int32_t *__restrict__ perm, int32_t *__restrict__ rank, double *__restrict__ ps,
    double *__restrict__ ms, uint64_t *__restrict__ qs, double *__restrict__ hs,
    int8_t *__restrict__ dR, uint32_t *__restrict__ base, uint32_t *__restrict__ sizes,
    uint32_t *__restrict__ bad_eps, uint32_t *hpin) {
    __shared__ uint64_t s_k[kSmallN];
    __shared__ uint32_t s_v[kSmallN];
    __shared__ uint32_t s_wc[kSmallWaves][256];
    __shared__ uint32_t s_loc[256], s_sc[kSmallWaves], s_lev[kLevels];
    __shared__ double s_red[6][kSmallWaves];
    __shared__ Frame s_F;
    __shared__ uint32_t s_bad;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int rounds = (n + kSmallBlock - 1) / kSmallBlock;  // a wavefront's keys: 64 a round
    const int wbase = w * rounds * 64;
    if (tid == 0)
        s_bad = 0u;
    if (tid < kLevels)
        s_lev[tid] = 0u;
    // 1. root cube
    if (!F0.periodic) {
        double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
        const double *c[3] = {x, y, z};
        for (int i = tid; i < n; i += kSmallBlock)
            for (int a = 0; a < 3; a++) {
                lo[a] = fmin(lo[a], c[a][i]);
                hi[a] = fmax(hi[a], c[a][i]);
            }
        for (int a = 0; a < 3; a++) {
            for (int o = 1; o < 64; o <<= 1) {
                lo[a] = fmin(lo[a], __shfl_xor(lo[a], o));
                hi[a] = fmax(hi[a], __shfl_xor(hi[a], o));
            }
            if (lane == 0) {
                s_red[a][w] = lo[a];
                s_red[3 + a][w] = hi[a];
            }
        }
        __syncthreads();
        if (tid == 0) {
            for (int a = 0; a < 3; a++)
                for (int q = 0; q < kSmallWaves; q++) {
                    lo[a] = fmin(lo[a], s_red[a][q]);
                    hi[a] = fmax(hi[a], s_red[3 + a][q]);
                }
            make_frame(lo, hi, s0, s1, s2, s_F);
        }
    } else if (tid == 0) {
        s_F = F0;
    }
    __syncthreads();
    const Frame F = s_F;
    // 2. keys
    uint64_t k[kSmallRounds];
    uint32_t v[kSmallRounds], pos[kSmallRounds];
#pragma unroll
    for (int r = 0; r < kSmallRounds; r++) {
        const int i = wbase + r * 64 + lane;
        k[r] = 0ull;
        v[r] = 0u;
        if (r < rounds && i < n) {
            double p;
            uint32_t q0, q1, q2;
            to_frame(x[i], F.x0[0], F, p, q0);
            to_frame(y[i], F.x0[1], F, p, q1);
            to_frame(z[i], F.x0[2], F, p, q2);
            k[r] = hilbert_key(q0, q1, q2);
            v[r] = (uint32_t)i;
        }
    }
    // 3. stable sort, eight 8-bit digits: the rank of a key is the number of
    // keys with smaller digits, of its digit in earlier wavefronts, and of its
    // digit before it in its wavefront's contiguous share
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    for (int shift = 0; shift < 64; shift += 8) {
        for (int q = tid; q < kSmallWaves * 256; q += kSmallBlock)
            (&s_wc[0][0])[q] = 0u;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSmallRounds; r++) {
            if (r >= rounds)
                break;
            const bool valid = wbase + r * 64 + lane < n;
            const uint32_t d = (uint32_t)(k[r] >> shift) & 255u;
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; b++) {
                const bool bit = (d >> b) & 1u;
                const uint64_t m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
            const uint32_t before = (uint32_t)__popcll(peers & lt);
            const uint32_t prev = s_wc[w][d];
            pos[r] = prev + before;
            __builtin_amdgcn_wave_barrier();
            if (valid && before == 0)
                s_wc[w][d] = prev + (uint32_t)__popcll(peers);
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        uint32_t cnt = 0u, inc = 0u;
        if (tid < 256) {
#pragma unroll
            for (int q = 0; q < kSmallWaves; q++) {
                const uint32_t cq = s_wc[q][tid];
                s_wc[q][tid] = cnt;
                cnt += cq;
            }
            inc = wave_scan(cnt, lane);
            if (lane == 63)
                s_sc[w] = inc;
        }
        __syncthreads();
        if (tid < 256) {
            uint32_t wb = 0u;
            for (int q = 0; q < w; q++)
                wb += s_sc[q];
            s_loc[tid] = wb + inc - cnt;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSmallRounds; r++) {
            if (r >= rounds)
                break;
            if (wbase + r * 64 + lane < n) {
                const uint32_t d = (uint32_t)(k[r] >> shift) & 255u;
                const uint32_t at = s_loc[d] + s_wc[w][d] + pos[r];
                s_k[at] = k[r];
                s_v[at] = v[r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSmallRounds; r++) {
            const int i = wbase + r * 64 + lane;
            if (r < rounds && i < n) {
                k[r] = s_k[i];
                v[r] = s_v[i];
            }
        }
        __syncthreads();
    }
    // 4. curve order; depths shared with the neighbours, entries per particle
    uint32_t run = 0u;  // entries of this wavefront's particles so far
#pragma unroll
    for (int r = 0; r < kSmallRounds; r++) {
        if (r >= rounds)
            break;
        const int s = wbase + r * 64 + lane;
        int dr = -1, dl = -1;
        if (s < n) {
            const uint32_t i = v[r];
            key[s] = k[r];
            perm[s] = (int32_t)i;
            rank[i] = s;
            double p0, p1, p2;
            uint32_t q0, q1, q2;
            to_frame(x[i], F.x0[0], F, p0, q0);
            to_frame(y[i], F.x0[1], F, p1, q1);
            to_frame(z[i], F.x0[2], F, p2, q2);
            ps[s] = p0;
            ps[(size_t)n + s] = p1;
            ps[2 * (size_t)n + s] = p2;
            ms[s] = mass ? mass[i] : 1.0 / (double)n;
            qs[s] = ((uint64_t)q0 << 42) | ((uint64_t)q1 << 21) | (uint64_t)q2;
            if (eps) {
                const double e = eps[i];
                if (!(e > 0.0) || !isfinite(e))
                    s_bad = 1u;
                hs[s] = 2.8 * e;
            }
            dr = s + 1 < n ? common_levels(k[r], s_k[s + 1]) : -1;
            dl = s > 0 ? common_levels(s_k[s - 1], k[r]) : -1;
            dR[s] = (int8_t)dr;
        }
        const uint32_t nn = dr > dl ? (uint32_t)(dr - dl) : 0u;
        const uint32_t c = s < n ? nn + 1u : 0u;
        const uint32_t in = wave_scan(c, lane);
        pos[r] = run + in - c;
        run += __shfl(in, 63);
        for (int lev = 0; lev < kLevels; lev++) {
            const uint32_t m = (uint32_t)__popcll(__ballot(lev > dl && lev <= dr));
            if (lane == 0 && m)
                atomicAdd(&s_lev[lev], m);
        }
    }
    if (lane == 0)
        s_sc[w] = run;
    __syncthreads();
    uint32_t wb = 0u, total = 0u;
    for (int q = 0; q < kSmallWaves; q++) {
        wb += q < w ? s_sc[q] : 0u;
        total += s_sc[q];
    }
#pragma unroll
    for (int r = 0; r < kSmallRounds; r++) {
        const int s = wbase + r * 64 + lane;
        if (r < rounds && s < n)
            base[s] = wb + pos[r];
    }
    if (tid == 0) {
        uint32_t at = 0u;
        for (int lev = 0; lev < kLevels; lev++) {
            sizes[lev] = hpin[lev] = at;
            at += s_lev[lev];
        }
        sizes[32] = hpin[32] = total;
        sizes[33] = hpin[33] = at;
        *Fp = F;
        *(Frame *)(hpin + 64) = F;
        if (s_bad)
            *bad_eps = 1u;
        hpin[128] = s_bad;
    }
}

__global__ __launch_bounds__(kSmallBlock) void k_small_back(
    int n, uint32_t E, const int8_t *__restrict__ dR, const uint32_t *__restrict__ base,
    const Frame *__restrict__ Fp, const uint32_t *__restrict__ sizes,
    const double *__restrict__ ps, const double *__restrict__ ms,
    const uint64_t *__restrict__ qs, Rec64 *rec, uint32_t *efirst, uint32_t *ecount, uint32_t *pe,
    uint32_t *lvl_list, const double *__restrict__ hs, double *eh, double G, Rec32 *out32,
    float *eh32) {
    // per entry: the entry after its subtree, and its depth
    __shared__ uint32_t s_skip[kSmallE];
    __shared__ uint8_t s_dep[kSmallE];
    __shared__ uint32_t s_cur[kLevels];
    const int tid = threadIdx.x;
    if (tid < kLevels)
        s_cur[tid] = sizes[tid];
    const Frame F = *Fp;
    __syncthreads();
    for (int s = tid; s < n; s += kSmallBlock) {
        const int r = dR[s], l = s > 0 ? (int)dR[s - 1] : -1;
        const uint32_t b = base[s];
        uint32_t q[3];
        emit_particle(s, n, l, r, r, b, F, ps, ms, qs, rec, efirst, ecount, pe, hs, eh, G, out32,
                      eh32, q);
        for (int lev = l + 1; lev <= r; lev++) {
            const uint32_t e = b + (uint32_t)(lev - l - 1);
            lvl_list[atomicAdd(&s_cur[lev], 1u)] = e;
            s_dep[e] = (uint8_t)lev;
        }
        const uint32_t ep = b + (uint32_t)(r > l ? r - l : 0);
        s_skip[ep] = ep + 1u;
        s_dep[ep] = (uint8_t)((r > l ? r : l) + 1);
    }
    __syncthreads();
    const int sh = F.periodic ? kRecShiftPer : kRecShiftIso;
    for (int lev = kMaxLevel; lev >= 0; lev--) {
        const uint32_t first = sizes[lev], last = s_cur[lev];
        if (first == last)
            continue;
        for (uint32_t i = first + (uint32_t)tid; i < last; i += kSmallBlock) {
            const uint32_t e = lvl_list[i];
            const Rec64 R = rec[e];
            const uint32_t f = efirst[e];
            const uint64_t qq = out32 ? qs[f] : 0ull;
            double M = 0.0, X0 = 0.0, X1 = 0.0, X2 = 0.0, hmax = 0.0;
            uint32_t k = e + 1u;
            for (;;) {  // eight children at a time: found in LDS, then loaded together
                uint32_t kid[8];
                int m = 0;
#pragma unroll
                for (int q = 0; q < 8; q++) {
                    const bool more = k < E && s_dep[k] > lev;
                    kid[q] = more ? k : e;
                    m += more ? 1 : 0;
                    k = more ? s_skip[k] : k;
                }
                double mk[8], c0[8], c1[8], c2[8], hk[8];
#pragma unroll
                for (int q = 0; q < 8; q++) {
                    const Rec64 *c = rec + kid[q];
                    mk[q] = c->mass;
                    c0[q] = c->com[0];
                    c1[q] = c->com[1];
                    c2[q] = c->com[2];
                    hk[q] = eh ? eh[kid[q]] : 0.0;
                }
#pragma unroll
                for (int q = 0; q < 8; q++)
                    if (q < m) {
                        hmax = hk[q] > hmax ? hk[q] : hmax;
                        M = M + mk[q];
                        X0 = fma(mk[q], c0[q], X0);
                        X1 = fma(mk[q], c1[q], X1);
                        X2 = fma(mk[q], c2[q], X2);
                    }
                if (m < 8)
                    break;
            }
            s_skip[e] = k;
            const uint32_t q[3] = {(uint32_t)(qq >> 42) & 0x1fffffu,
                                   (uint32_t)(qq >> 21) & 0x1fffffu, (uint32_t)qq & 0x1fffffu};
            finish_node(rec, e, k, (k < E ? efirst[k] : (uint32_t)n) - f, (uint32_t)lev, R, M, X0,
                        X1, X2, hmax, q, ecount, eh, G, sh, out32, eh32);
        }
        __syncthreads();
    }
}

}  // namespace

size_t topology_hist_bytes(int64_t n) {
    return (size_t)2 * kLevels * grid_for(n, kBlock) * sizeof(uint32_t);
}

size_t bbox_bytes(int64_t n) {
    return (size_t)std::min<int64_t>(1024, (n + kBlock - 1) / kBlock) * 6 * sizeof(double);
}

// The level lists' offsets from the sizes read back.
static void set_levels(tpm_ctx *c) {
    for (int l = 0; l < kLevels; l++)
        c->level_off[l] = c->hpin[l];
    c->level_off[kLevels] = c->hpin[33];
    for (int l = 0; l < kLevels; l++)
        c->level_count[l] = c->level_off[l + 1] - c->level_off[l];
}

int build(tpm_ctx *c, int64_t n, const double *x, const double *y, const double *z,
          const double *mass, const double *eps) {
    hipStream_t st = c->stream;
    const tpm_params &P = c->P;
    // per-particle buffers
    TPM_TRY(ensure(c, c->frame, sizeof(Frame)));
    for (int b = 0; b < 2; b++) {
        TPM_TRY(ensure(c, c->key[b], (size_t)n * 8));
        TPM_TRY(ensure(c, c->idx[b], (size_t)n * 4));
    }
    TPM_TRY(ensure(c, c->perm, (size_t)n * 4));
    TPM_TRY(ensure(c, c->xyzm, (size_t)n * 32));
    TPM_TRY(ensure(c, c->rank, (size_t)n * 4));
    TPM_TRY(ensure(c, c->ps, (size_t)n * 24));
    TPM_TRY(ensure(c, c->ms, (size_t)n * 8));
    TPM_TRY(ensure(c, c->qs, (size_t)n * 8));
    TPM_TRY(ensure(c, c->dR, (size_t)n));
    TPM_TRY(ensure(c, c->cnt, (size_t)n * 4));
    TPM_TRY(ensure(c, c->base, (size_t)n * 4));
    TPM_TRY(ensure(c, c->pe, (size_t)n * 4));
    TPM_TRY(ensure(c, c->counters, 64 * sizeof(uint32_t)));
    TPM_TRY(ensure(c, c->lvl_cursor, 32 * sizeof(uint32_t)));
    Frame *F = (Frame *)c->frame.p;
    const uint64_t *key = (const uint64_t *)c->key[0].p;

    uint32_t *lvl_count = (uint32_t *)c->counters.p;  // [0..21] level starts, [32] E, [33] nodes
    uint32_t *bad_eps = (uint32_t *)c->err_flag.p + 1;
    const uint32_t nb = grid_for(n, kBlock);
    uint32_t *loff = nullptr;
    // individual softening: spline supports in curve order; a bad value
    // sets the second error word, read back with the sizes below
    c->mixed = eps != nullptr;
    if (c->mixed)
        TPM_TRY(ensure(c, c->hs, (size_t)n * 8));
    Frame h{};
    if (P.periodic) {
        for (int a = 0; a < 3; a++)
            h.x0[a] = -(P.shift[a] * P.box_size);
        h.L = P.box_size;
        h.S = 2097152.0 / P.box_size;
        h.box = P.box_size;
        h.periodic = 1;
    }
    const bool small = n <= kSmallN;
    if (small) {
        TPM_TRY(timer_begin(c, TPM_TIMER_TOPOLOGY));
        k_small_front<<<1, kSmallBlock, 0, st>>>(
            x, y, z, mass, eps, (int)n, h, P.shift[0], P.shift[1], P.shift[2], F,
            (uint64_t *)c->key[0].p, (int32_t *)c->perm.p, (int32_t *)c->rank.p,
            (double *)c->ps.p, (double *)c->ms.p, (uint64_t *)c->qs.p, (double *)c->hs.p,
            (int8_t *)c->dR.p, (uint32_t *)c->base.p, lvl_count, bad_eps, c->hpin_dev);
        TPM_LAUNCHED(c, "k_small_front");
        TPM_TRY(timer_end(c, TPM_TIMER_TOPOLOGY));
    } else {
    // 1. root cube
    TPM_TRY(timer_begin(c, TPM_TIMER_KEYS));
    if (P.periodic) {
        k_set_frame<<<1, 1, 0, st>>>(h, F);
        TPM_LAUNCHED(c, "k_set_frame");
    } else {
        const int nparts = (int)std::min<int64_t>(1024, (n + kBlock - 1) / kBlock);
        TPM_TRY(ensure(c, c->bbox, bbox_bytes(n)));
        k_bbox_partial<<<nparts, kBlock, 0, st>>>(x, y, z, n, (double *)c->bbox.p);
        TPM_LAUNCHED(c, "k_bbox_partial");
        k_frame_final<<<1, kBlock, 0, st>>>((const double *)c->bbox.p, nparts, F, P.shift[0],
                                            P.shift[1], P.shift[2]);
        TPM_LAUNCHED(c, "k_frame_final");
    }
    // 2. keys, 3. sort, gather
    k_keys<<<grid_for(n, kBlock), kBlock, 0, st>>>(x, y, z, mass, n, F,
                                                   (uint64_t *)c->key[0].p,
                                                   (uint32_t *)c->idx[0].p, (double4 *)c->xyzm.p);
    TPM_LAUNCHED(c, "k_keys");
    TPM_TRY(timer_end(c, TPM_TIMER_KEYS));
    TPM_TRY(radix_sort_pairs(c, n));
    TPM_TRY(timer_begin(c, TPM_TIMER_GATHER));
    k_gather<<<grid_for(n, kBlock), kBlock, 0, st>>>(
        (const double4 *)c->xyzm.p, n, F, (const uint32_t *)c->idx[0].p, (int32_t *)c->perm.p,
        (int32_t *)c->rank.p, (double *)c->ps.p, (double *)c->ms.p, (uint64_t *)c->qs.p, eps,
        c->mixed ? (double *)c->hs.p : nullptr, bad_eps);
    TPM_LAUNCHED(c, "k_gather");
    TPM_TRY(timer_end(c, TPM_TIMER_GATHER));
    // 4. topology: counts, scan, one readback of the sizes
    TPM_TRY(ensure(c, c->hist, topology_hist_bytes(n)));
    uint32_t *lhist = (uint32_t *)c->hist.p;
    loff = lhist + (size_t)kLevels * nb;
    TPM_TRY(timer_begin(c, TPM_TIMER_TOPOLOGY));
    k_count<<<nb, kBlock, 0, st>>>(key, n, (int8_t *)c->dR.p, (uint32_t *)c->cnt.p, lhist, nb);
    TPM_LAUNCHED(c, "k_count");
    TPM_TRY(scan_u32(c, (const uint32_t *)c->cnt.p, (uint32_t *)c->base.p, n, lvl_count + 32));
    TPM_TRY(scan_u32(c, lhist, loff, (int64_t)kLevels * nb, lvl_count + 33));
    k_sizes<<<1, 64, 0, st>>>(loff, nb, lvl_count + 32, F, bad_eps, c->hpin_dev);
    TPM_LAUNCHED(c, "k_sizes");
    TPM_TRY(timer_end(c, TPM_TIMER_TOPOLOGY));
    }
    TPM_HIP(c, hipStreamSynchronize(st));
    std::memcpy(&c->frame_host, c->hpin + 64, sizeof(Frame));
    if (c->hpin[128]) {
        TPM_TRY(fill_u32(c, bad_eps, 0u, 1));
        return fail(c, TPM_EINVAL, "softening lengths must be positive and finite");
    }
    // the FP32 walk works in units of L 2^-22 and scales sizes by 2^-level
    // through the exponent: both need a root size well inside float range
    if (P.precision == TPM_FP32 &&
        !(c->frame_host.L >= 0x1p-80 && c->frame_host.L <= 0x1p+80))
        return fail(c, TPM_EINVAL, "FP32 path: root cube size outside [2^-80, 2^80]");
    const uint32_t E = c->hpin[32];
    const uint32_t nodes = c->hpin[33];  // in the level lists
    if (E < (uint64_t)n || (uint64_t)E - (uint64_t)n < nodes)
        return fail(c, TPM_EDEVICE, "tree build: entry count mismatch");
    set_levels(c);
    const uint32_t off = nodes;
    TPM_TRY(ensure(c, c->rec64, (size_t)E * sizeof(Rec64)));
    TPM_TRY(ensure(c, c->efirst, (size_t)E * 4));
    TPM_TRY(ensure(c, c->ecount, (size_t)E * 4));
    TPM_TRY(ensure(c, c->lvl_list, (size_t)(off > 0 ? off : 1) * 4));
    Rec64 *rec = (Rec64 *)c->rec64.p;
    // FP32 records: particles' written by the emission, nodes' by the moments
    Rec32 *rec32 = nullptr;
    float *eh32 = nullptr;
    if (P.precision == TPM_FP32) {
        TPM_TRY(ensure(c, c->rec32, (size_t)E * sizeof(Rec32)));
        rec32 = (Rec32 *)c->rec32.p;
        if (c->mixed) {
            TPM_TRY(ensure(c, c->eh32, (size_t)E * 4));
            eh32 = (float *)c->eh32.p;
        }
    }
    double *eh = nullptr;
    if (c->mixed) {
        TPM_TRY(ensure(c, c->eh64, (size_t)E * 8));
        eh = (double *)c->eh64.p;
    }
    if (small && E <= kSmallE) {
        TPM_TRY(timer_begin(c, TPM_TIMER_MOMENTS));
        k_small_back<<<1, kSmallBlock, 0, st>>>(
            (int)n, E, (const int8_t *)c->dR.p, (const uint32_t *)c->base.p, F, lvl_count,
            (const double *)c->ps.p, (const double *)c->ms.p, (const uint64_t *)c->qs.p, rec,
            (uint32_t *)c->efirst.p, (uint32_t *)c->ecount.p, (uint32_t *)c->pe.p,
            (uint32_t *)c->lvl_list.p, (const double *)c->hs.p, eh, P.G, rec32, eh32);
        TPM_LAUNCHED(c, "k_small_back");
        TPM_TRY(timer_end(c, TPM_TIMER_MOMENTS));
        c->n = n;
        c->E = E;
        return TPM_OK;
    }
    if (small) {  // too many entries for its LDS: the general kernels' level offsets
        TPM_TRY(ensure(c, c->hist, topology_hist_bytes(n)));
        uint32_t *lhist = (uint32_t *)c->hist.p;
        loff = lhist + (size_t)kLevels * nb;
        k_count<<<nb, kBlock, 0, st>>>(key, n, (int8_t *)c->dR.p, (uint32_t *)c->cnt.p, lhist,
                                       nb);
        TPM_LAUNCHED(c, "k_count");
        TPM_TRY(scan_u32(c, lhist, loff, (int64_t)kLevels * nb, lvl_count + 33));
        k_sizes<<<1, 64, 0, st>>>(loff, nb, lvl_count + 32, F, bad_eps, c->hpin_dev);
        TPM_LAUNCHED(c, "k_sizes");
        TPM_HIP(c, hipStreamSynchronize(st));
        set_levels(c);
    }
    TPM_TRY(timer_begin(c, TPM_TIMER_TOPOLOGY));
    auto emit = c->mixed ? k_emit<true> : k_emit<false>;
    emit<<<grid_for(n, kBlock), kBlock, 0, st>>>(
        n, E, (const int8_t *)c->dR.p, (const uint32_t *)c->base.p, F, (const double *)c->ps.p,
        (const double *)c->ms.p, (const uint64_t *)c->qs.p, rec, (uint32_t *)c->efirst.p,
        (uint32_t *)c->ecount.p, (uint32_t *)c->pe.p, loff, nb, (uint32_t *)c->lvl_list.p,
        (const double *)c->hs.p, eh, P.G, rec32, eh32);
    TPM_LAUNCHED(c, "k_emit");
    TPM_TRY(timer_end(c, TPM_TIMER_TOPOLOGY));
    // 5. moments, deepest level first
    TPM_TRY(timer_begin(c, TPM_TIMER_MOMENTS));
    LevelOffsets lo;
    std::memcpy(lo.off, c->level_off, sizeof lo.off);
    const int sh = P.periodic ? kRecShiftPer : kRecShiftIso;
    for (int l = kMaxLevel; l >= 0;) {
        int top = l;  // levels top .. l: one launch
        uint32_t most = c->level_count[l];
        while (most <= kRunNodes && top > 0 && c->level_count[top - 1] <= kRunNodes)
            most = std::max(most, c->level_count[--top]);
        if (most > kRunNodes) {
            const uint32_t cnt = c->level_count[l];
            k_moments<<<grid_for(cnt, kBlock), kBlock, 0, st>>>(
                rec, E, (uint32_t)n, (const uint32_t *)c->efirst.p, (uint32_t *)c->ecount.p,
                (const uint32_t *)c->lvl_list.p + c->level_off[l], cnt, (uint32_t)l, eh, P.G,
                (const uint64_t *)c->qs.p, sh, rec32, eh32);
            TPM_LAUNCHED(c, "k_moments");
        } else if (most > 0) {
            k_moments_run<<<1, kRunNodes, 0, st>>>(
                rec, E, (uint32_t)n, (const uint32_t *)c->efirst.p, (uint32_t *)c->ecount.p,
                (const uint32_t *)c->lvl_list.p, lo, l, top, eh, P.G, (const uint64_t *)c->qs.p,
                sh, rec32, eh32);
            TPM_LAUNCHED(c, "k_moments_run");
        }
        l = top - 1;
    }
    TPM_TRY(timer_end(c, TPM_TIMER_MOMENTS));
    c->n = n;
    c->E = E;
    return TPM_OK;
}

}  // namespace tpm
