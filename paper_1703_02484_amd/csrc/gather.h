// Sums over the chunks of a disk's per-chunk partial sums, shared by the update, the force read-out and the adjoint
// sweep.  A chunk holds one species and a system's chunks are in species order.
//
// Bound by latency: a disk's partial sums lie a system apart, so a wavefront has one load per chunk and nothing else
// to do.  Sixteen loads go out before their sums; the chunk list is read by the scalar unit (one system at a time:
// the list is then the same for every lane), and the strength multiplies a species' sum, not each chunk's.  Handles
// of many chunks give each group of 64 disks W wavefronts, a part of the chunks each, added in LDS in order.
#pragma once

#include "bd_internal.h"

namespace bd {

// Handles of up to kGatherSmall disks run 64 to a workgroup, which spreads them over more compute units; from
// kGatherSplit chunks on with four wavefronts.  The update of 16,384 disks (128 chunks, FP64): 11 us with four, 12.6
// with one, 20 us with one and the chunk list read per lane; 16,001 (63 chunks) 7.4, 8.7 and 13.7.  Larger handles
// have wavefronts enough and are bound by the bytes: 65,536 (128 chunks, FP32) 18.3 us with one, 20.4 with four.
constexpr int kGatherSmall = 32768;
constexpr int kGatherSplit = 32;

// Sums chunks [c0, c1) at `row` and calls flush(species, x, y) after each run of chunks of one species.  Everything
// but part and row is the same for every lane.
template <typename T2, class F>
__device__ __forceinline__ void gather_chunks(const T2 *__restrict__ part, long long row, int stride,
                                              const int *__restrict__ spec, int c0, int c1, F &&flush) {
    constexpr int kB = 16;
    if (c0 >= c1) return;
    int b = spec[c0];
    double sx = 0.0, sy = 0.0;
    for (int c = c0; c < c1; c += kB) {
        T2 v[kB];
#pragma unroll
        for (int u = 0; u < kB; ++u) {   // past the end: the last one again, not added
            const int cu = c + u < c1 ? c + u : c1 - 1;
            v[u] = part[row + (long long)cu * stride];
        }
        const int m = c1 - c < kB ? c1 - c : kB;
        if (m == kB && spec[c + kB - 1] == b) {
#pragma unroll
            for (int u = 0; u < kB; ++u) {
                sx += (double)v[u].x;
                sy += (double)v[u].y;
            }
            continue;
        }
#pragma unroll
        for (int u = 0; u < kB; ++u) {
            if (u < m) {
                const int bu = spec[c + u];
                if (bu != b) {
                    flush(b, sx, sy);
                    sx = sy = 0.0;
                    b = bu;
                }
                sx += (double)v[u].x;
                sy += (double)v[u].y;
            }
        }
    }
    flush(b, sx, sy);
}

// Calls f(system) once for each system among the active lanes, with the lanes of that system.  The loop's condition
// is the same for every lane (a lane that left by itself would run f after the loop, together with the others).
template <class F>
__device__ __forceinline__ void each_system(int rep, F &&f) {
    for (unsigned long long rest = __ballot(true); rest != 0;) {
        const bool mine = rep == __builtin_amdgcn_readlane(rep, __ffsll(rest) - 1);
        if (mine) f(__builtin_amdgcn_readfirstlane(rep));   // read again: known as one value for these lanes
        rest &= ~__ballot(mine);
    }
}

// Whether 64 disks take four wavefronts.
inline bool gather_split(const Sim &s) { return s.n <= kGatherSmall && s.nch_max >= kGatherSplit; }

// F_i = sum_b K[s_i][b] sum_{c in b} Phi_{i,c}, FP64; k is i's sorted index.  The chunks of a system of kGatherSplit
// or more are summed in four parts, the parts then in order, whoever sums them: a system's forces do not depend on
// what else its handle holds.  W (1 or 4) wavefronts per 64 disks: every thread calls it (valid: there is a disk for
// this lane), and the result is wavefront 0's.
template <typename T2, int W>
__device__ __forceinline__ void gather_force(const T2 *__restrict__ part, const RepInfo *__restrict__ reps, int rep,
                                             const int *__restrict__ chunk_spec, const double *__restrict__ K, int S,
                                             int si, int k, bool valid, double &fx, double &fy) {
    __shared__ double2 sum[W > 1 ? W - 1 : 1][64];
    const int w = W > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) : 0;
    fx = fy = 0.0;
    if (valid)
        each_system(rep, [&](int r) {
            const RepInfo ri = reps[r];
            const int parts = ri.nch >= kGatherSplit ? 4 : 1;
            for (int p = w; p < parts; p += W) {
                double gx = 0.0, gy = 0.0;
                gather_chunks(part, ri.poff + (k - ri.off), ri.n, chunk_spec + ri.cfirst, ri.nch * p / parts,
                              ri.nch * (p + 1) / parts, [&](int b, double sx, double sy) {
                                  const double kab = K[si * S + b];
                                  gx += kab * sx;
                                  gy += kab * sy;
                              });
                fx += gx;
                fy += gy;
            }
        });
    if (W == 1) return;
    if (w > 0) sum[w - 1][threadIdx.x & 63] = make_double2(fx, fy);
    __syncthreads();
    if (w > 0) return;
#pragma unroll
    for (int u = 0; u < W - 1; ++u) {
        const double2 a = sum[u][threadIdx.x];
        fx += a.x;
        fy += a.y;
    }
}

}  // namespace bd
