// Adjoint (reverse-mode) sweep of the time step: gradients of a loss on the
// final positions with respect to the initial positions and the strength
// matrix K.  Not part of the paper's method.  The step is differentiated as
// written with every discrete choice of the forward pass held fixed: the
// overlapping partners of each correction round (the correction acts as a
// projection onto that round's contact set), the cap branch and the wall
// branches.  Noise and the director angles do not depend on the positions.
//
// Per step, in reverse (lambda = dL/dx after the step):
//   overlap rounds, last first: mu = S_w lambda (wall slopes), nu = C^T mu
//     (cap: (c/|D|)(I - e e^T) when the cap acted), then for a moved disk m
//     lambda_m = mu_m + sum_{j overlapping m} A_mj (nu_m - nu_j),
//     A = f((sigma/d - 1) I - (sigma/d) n n^T) at the positions before the round;
//   the move x* = x + dt F(x) + noise, then walls:
//     lambda* = S_w lambda,
//     dL/dK[a][b] += dt sum_{i in a} lambda*_i . Phi_{i,b},  Phi_{i,b} = sum_{j in b} u_ij / d^3,
//     lambda = lambda* + dt g,  g_m = sum_j J(u_mj) (K[s_m][s_j] lambda*_m - K[s_j][s_m] lambda*_j),
//     J(u) = (I - 3 n n^T) / d^3 for the inverse-square law.
// g is an all-pairs sum like the force; it runs over the force's tiles and
// is reduced per particle in a fixed chunk order, so the sweep is
// deterministic.
#include <hip/hip_runtime.h>

#include "gather.h"
#include "geom.h"

namespace bd {
namespace {

constexpr int kAdjBlock = 256;

// ---------------------------------------------------------------- overlap rounds
// What the tape holds of one moved disk in one round.
struct RoundEntry {
    int v, na;            // the disk; its overlapping partners
    int4 nb;              // the first four of them
    double sx, sy, r;     // wall slopes, radius
    double2 old, disp;    // position before the round, uncapped sum
};

struct RoundTape {
    const int *ev;
    const double2 *eold, *edisp;
    const signed char *ewf;
    const int *ecnt, *enb;
    const double *rad;
    double cap_frac, f;
};

__device__ __forceinline__ RoundEntry round_entry(const RoundTape &t, int e) {
    RoundEntry q;
    q.v = t.ev[e];
    q.na = t.ecnt[e];
    q.nb = *(const int4 *)(t.enb + (size_t)e * MAXACT);
    q.sx = t.ewf[2 * (size_t)e];
    q.sy = t.ewf[2 * (size_t)e + 1];
    q.old = t.eold[e];
    q.disp = t.edisp[e];
    q.r = t.rad[q.v];
    return q;
}

// mu = S_w lambda, nu = C^T mu; nub holds nu and the position before the round, by disk.
__device__ __forceinline__ void round_prep(const RoundTape &t, const RoundEntry &q, double2 l, double4 *nub) {
#pragma clang fp contract(off)
    double mx = q.sx * l.x, my = q.sy * l.y;
    const double2 D = q.disp;
    const double len = sqrt(D.x * D.x + D.y * D.y);
    const double cap = t.cap_frac * q.r;
    if (len > cap) {
        const double ex = D.x / len, ey = D.y / len, sc = cap / len;
        const double em = ex * mx + ey * my;
        mx = sc * (mx - ex * em);
        my = sc * (my - ey * em);
    }
    nub[q.v] = make_double4(mx, my, q.old.x, q.old.y);
}

__device__ __forceinline__ double2 round_apply(const RoundTape &t, const RoundEntry &q, int e, double2 l,
                                               const double4 *nub) {
#pragma clang fp contract(off)
    double ax = q.sx * l.x, ay = q.sy * l.y;
    const double4 nv = nub[q.v];
    for (int k0 = 0; k0 < q.na; k0 += 4) {
        const int4 nb = k0 == 0 ? q.nb : *(const int4 *)(t.enb + (size_t)e * MAXACT + k0);
        const int id[4] = {nb.x, nb.y, nb.z, nb.w};
        double4 nj[4];
        double rj[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = k0 + u < q.na ? id[u] : q.v;
            nj[u] = nub[j];
            rj[u] = t.rad[j];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (k0 + u >= q.na) break;
            const double ux = nv.z - nj[u].z, uy = nv.w - nj[u].w;
            const double d = sqrt(ux * ux + uy * uy);
            const double nx = ux / d, ny = uy / d;
            const double a = (q.r + rj[u]) / d;
            const double dx = nv.x - nj[u].x, dy = nv.y - nj[u].y;
            const double nd = nx * dx + ny * dy;
            ax += t.f * ((a - 1.0) * dx - a * nx * nd);
            ay += t.f * ((a - 1.0) * dy - a * ny * nd);
        }
    }
    return make_double2(ax, ay);
}

// One large round as two launches.
__global__ void k_adj_round_prep(int e0, int cnt, RoundTape t, const double2 *__restrict__ lam,
                                 double4 *__restrict__ nub) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= cnt) return;
    const RoundEntry q = round_entry(t, e0 + idx);
    round_prep(t, q, lam[q.v], nub);
}

__global__ void k_adj_round_apply(int e0, int cnt, RoundTape t, const double4 *__restrict__ nub,
                                  double2 *__restrict__ lam) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= cnt) return;
    const RoundEntry q = round_entry(t, e0 + idx);
    lam[q.v] = round_apply(t, q, e0 + idx, lam[q.v], nub);
}

// Rounds [r0, r1), last first, in one workgroup with a barrier between their halves: a round is a chain of a few
// loads, shorter than a launch.  A thread's entry of the next round is loaded while this one is applied (the tape
// does not change), so a round waits for lambda and nu only.  Rounds above kAdjRoundMax entries are launched by
// themselves, where many compute units share them.  16,384 disks, some 18 rounds of up to 500 entries a step: 160 us
// in launches of their own, 37 us so.
constexpr int kRoundsBlock = 1024;
constexpr int kAdjRoundMax = 4 * kRoundsBlock;

__global__ __launch_bounds__(kRoundsBlock) void k_adj_rounds(const int2 *__restrict__ dir, int r0, int r1, RoundTape t,
                                                             double2 *lam, double4 *nub) {
    const int tid = threadIdx.x;
    int2 d = dir[r1 - 1];
    RoundEntry q{};
    if (tid < d.y) q = round_entry(t, d.x + tid);
    for (int r = r1 - 1; r >= r0; --r) {
        const int2 next = r > r0 ? dir[r - 1] : make_int2(0, 0);
        double2 l = make_double2(0.0, 0.0);
        if (tid < d.y) {
            l = lam[q.v];
            round_prep(t, q, l, nub);
        }
        for (int idx = tid + kRoundsBlock; idx < d.y; idx += kRoundsBlock) {
            const RoundEntry o = round_entry(t, d.x + idx);
            round_prep(t, o, lam[o.v], nub);
        }
        __syncthreads();
        RoundEntry qn{};
        if (tid < next.y) qn = round_entry(t, next.x + tid);
        if (tid < d.y) lam[q.v] = round_apply(t, q, d.x + tid, l, nub);
        for (int idx = tid + kRoundsBlock; idx < d.y; idx += kRoundsBlock) {
            const RoundEntry o = round_entry(t, d.x + idx);
            lam[o.v] = round_apply(t, o, d.x + idx, lam[o.v], nub);
        }
        __syncthreads();
        q = qn;
        d = next;
    }
}

// ---------------------------------------------------------------- the move
// lambda* = S_w lambda, and sorted copies of the positions before the step: (x, y, lambda*) in FP64 for the adjoint
// pair sum, and where pj is given the force kernel's own copy to recompute Phi.
template <typename T2>
__global__ void k_adj_cast(int n, const double *__restrict__ px, const double *__restrict__ py,
                           const signed char *__restrict__ wf, const int *__restrict__ sorted_id,
                           double2 *__restrict__ lam, double4 *__restrict__ pj4, T2 *__restrict__ pj) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int i = sorted_id[k];
    const double x = px[i], y = py[i];
    double2 l = lam[i];
    l = make_double2(wf[2 * (size_t)i] * l.x, wf[2 * (size_t)i + 1] * l.y);
    lam[i] = l;
    pj4[k] = make_double4(x, y, l.x, l.y);
    if (!pj) return;
    T2 v;
    v.x = x;
    v.y = y;
    pj[k] = v;
}

// The end of a step's move, for 64 disks by four wavefronts, each a part of the chunks (gather.h):
//   dL/dK[a][b] += dt sum_{i in a} lambda*_i . Phi_{i,b}, the sum over the disks in a fixed order per (a, b), added
//   to the workgroup's own accumulator, so the result does not depend on scheduling;
//   lambda = lambda* + dt g, g reduced over the disk's chunks in a fixed order.
// 16,384 disks in 128 chunks: 14 us; 142 us as three launches of one thread per disk or per (block, a, b).
constexpr int kUpdateWaves = 4;

template <typename T2>
__global__ __launch_bounds__(64 * kUpdateWaves) void k_adj_update(
    int n, int S, const T2 *__restrict__ phi, const double2 *__restrict__ gpart, const RepInfo *__restrict__ reps,
    const int *__restrict__ rep_of, const int *__restrict__ chunk_spec, const int *__restrict__ sp,
    const int *__restrict__ pos_of, double dt, double2 *__restrict__ lam, double *__restrict__ dk_blk) {
    __shared__ double rows[kUpdateWaves][BD_MAX_SPECIES][64];
    __shared__ double2 gsum[kUpdateWaves][64];
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = blockIdx.x * 64 + lane;
    const bool valid = i < n;
    const double2 l = valid ? lam[i] : make_double2(0.0, 0.0);
    for (int b = 0; b < S; ++b) rows[w][b][lane] = 0.0;
    double gx = 0.0, gy = 0.0;
    if (valid)
        each_system(rep_of[i], [&](int r) {
            const RepInfo ri = reps[r];
            const long long row = ri.poff + (pos_of[i] - ri.off);
            const int c0 = ri.nch * w / kUpdateWaves, c1 = ri.nch * (w + 1) / kUpdateWaves;
            const int *spec = chunk_spec + ri.cfirst;
            gather_chunks(phi, row, ri.n, spec, c0, c1, [&](int b, double sx, double sy) {
                rows[w][b][lane] += dt * (l.x * sx + l.y * sy);
            });
            gather_chunks(gpart, row, ri.n, spec, c0, c1, [&](int, double sx, double sy) {
                gx += sx;
                gy += sy;
            });
        });
    gsum[w][lane] = make_double2(gx, gy);
    __syncthreads();
    if (w == 0 && valid) {
        double2 g = gsum[0][lane];
        for (int u = 1; u < kUpdateWaves; ++u) {
            g.x += gsum[u][lane].x;
            g.y += gsum[u][lane].y;
        }
        lam[i] = make_double2(l.x + dt * g.x, l.y + dt * g.y);
    }
    const int si = valid ? sp[i] : -1;
    for (int ab = w; ab < S * S; ab += kUpdateWaves) {
        const int a = ab / S, b = ab % S;
        double v = 0.0;
        if (si == a)
            for (int u = 0; u < kUpdateWaves; ++u) v += rows[u][b][lane];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if (lane == 0) dk_blk[(size_t)blockIdx.x * S * S + ab] += v;
    }
}

// One workgroup per (a, b).
__global__ __launch_bounds__(kAdjBlock) void k_adj_dk_final(int nblk, int S, const double *__restrict__ dk_blk,
                                                            double *__restrict__ dk) {
    __shared__ double sum[kAdjBlock];
    double s = 0.0;
    for (int b = threadIdx.x; b < nblk; b += kAdjBlock) s += dk_blk[(size_t)b * S * S + blockIdx.x];
    sum[threadIdx.x] = s;
    for (int h = kAdjBlock / 2; h > 0; h >>= 1) {
        __syncthreads();
        if (threadIdx.x < h) sum[threadIdx.x] += sum[threadIdx.x + h];
    }
    if (threadIdx.x == 0) dk[blockIdx.x] = sum[0];
}

// Adjoint pair sum over one tile: for each i of the tile and the chunk's
// species b, M = sum_j J(u_ij) and v = sum_j J(u_ij) lambda*_j, then
// gpart = K[s_i][b] M lambda*_i - K[b][s_i] v.
template <int P, bool SELF>
__device__ __forceinline__ void adj_range(const double4 *__restrict__ pj4, int j0, int j1, int ib,
                                          const double (&xi)[P], const double (&yi)[P], double (&mxx)[P],
                                          double (&mxy)[P], double (&myy)[P], double (&vx)[P],
                                          double (&vy)[P]) {
    for (int j = j0; j < j1; ++j) {
        const double4 q = pj4[j];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            if (SELF && j == ib + k * kAdjBlock + (int)threadIdx.x) continue;
            const double ux = xi[k] - q.x, uy = yi[k] - q.y;
            const double d2 = ux * ux + uy * uy;
            // d^-1 from the hardware estimate y0, corrected with e = 1 - d2 y0^2:
            // y0 (1 - e)^-1/2 ~ y0 (1 + e/2 + 3/8 e^2), relative error O(e^3)
            const double y0 = __builtin_amdgcn_rsq(d2);
            const double e = fma(-d2, y0 * y0, 1.0);
            const double inv = y0 * fma(fma(0.375, e, 0.5), e, 1.0);
            const double inv2 = inv * inv;
            const double inv3 = inv2 * inv;
            const double c5 = 3.0 * inv3 * inv2;
            const double tx = c5 * ux, ty = c5 * uy;
            const double jxx = inv3 - tx * ux;
            const double jxy = -tx * uy;
            const double jyy = inv3 - ty * uy;
            mxx[k] += jxx;
            mxy[k] += jxy;
            myy[k] += jyy;
            vx[k] += jxx * q.z + jxy * q.w;
            vy[k] += jxy * q.z + jyy * q.w;
        }
    }
}

template <int P>
__global__ __launch_bounds__(kAdjBlock) void k_adj_pairs(const double4 *__restrict__ pj4,
                                                         const int *__restrict__ sps, const Tile *__restrict__ tiles,
                                                         const double *__restrict__ K, int S,
                                                         double2 *__restrict__ gpart) {
    const Tile tl = tiles[blockIdx.x];
    const int ib = tl.i0;
    double xi[P], yi[P], mxx[P], mxy[P], myy[P], vx[P], vy[P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const int i = ib + k * kAdjBlock + threadIdx.x;
        const double4 v = pj4[i < tl.i1 ? i : tl.i1 - 1];
        xi[k] = v.x;
        yi[k] = v.y;
        mxx[k] = mxy[k] = myy[k] = vx[k] = vy[k] = 0.0;
    }
    const int lo = tl.js > ib ? tl.js : ib;
    const int hi = tl.je < tl.i1 ? tl.je : tl.i1;
    if (lo < hi) {
        adj_range<P, false>(pj4, tl.js, lo, ib, xi, yi, mxx, mxy, myy, vx, vy);
        adj_range<P, true>(pj4, lo, hi, ib, xi, yi, mxx, mxy, myy, vx, vy);
        adj_range<P, false>(pj4, hi, tl.je, ib, xi, yi, mxx, mxy, myy, vx, vy);
    } else {
        adj_range<P, false>(pj4, tl.js, tl.je, ib, xi, yi, mxx, mxy, myy, vx, vy);
    }
    const int b = sps[tl.js];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const int i = ib + k * kAdjBlock + threadIdx.x;
        if (i < tl.i1) {
            const double4 v = pj4[i];
            const int si = sps[i];
            const double kab = K[si * S + b], kba = K[b * S + si];
            const double gx = kab * (mxx[k] * v.z + mxy[k] * v.w) - kba * vx[k];
            const double gy = kab * (mxy[k] * v.z + myy[k] * v.w) - kba * vy[k];
            gpart[tl.pbase + i] = make_double2(gx, gy);
        }
    }
}

// The same sum over unordered pairs, for the symmetric force's chunk pairs (A, B) of species a, b: with
// w = K[a][b] lambda*_i - K[b][a] lambda*_j the pair adds J w to i's sum and takes it from j's,
// J w = d^-3 (w - 3 d^-2 (u . w) u).  The turning of j around the wavefront, the LDS copy of the j sums, the padding
// (at +-BIG: d^-3 underflows to exactly 0) and the layout of the result are those of the force; a chunk paired with
// itself takes i's side only and leaves out i == j.
// VALU-bound: 27 FP64 instructions (1.2 issue slots each), v_rsq_f64 (4.3) and 12 / P DPP moves per unordered pair
// against 2 x 29 and 2 x 4.3 with both orders.  FP64, 16,384 disks: 152 us, 270 us ordered.
constexpr double kAdjBig = 1e150;

__device__ __forceinline__ double rot1d(double v) {   // lane l takes lane l + 1's value
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffll), 0x134, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x134, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// 64 steps of one group of 64 j, this lane's being j; SELF: at step t, lane i of vector p meets itself when same == p
// and t == 0.
template <int P, bool SELF>
__device__ __forceinline__ void adj_group(const double (&xi)[P], const double (&yi)[P], const double (&ax)[P],
                                          const double (&ay)[P], double (&gx)[P], double (&gy)[P], double xj, double yj,
                                          double bx, double by, double &hx, double &hy, int same) {
    for (int t = 0; t < 64; ++t) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const double ux = xi[p] - xj, uy = yi[p] - yj;
            const double d2 = ux * ux + uy * uy;
            double y0 = __builtin_amdgcn_rsq(d2);   // corrected as in adj_range
            if (SELF) y0 = t == 0 && same == p ? 0.0 : y0;
            const double e = fma(-d2, y0 * y0, 1.0);
            const double inv = y0 * fma(fma(0.375, e, 0.5), e, 1.0);
            const double inv2 = inv * inv;
            const double inv3 = inv2 * inv;
            const double wx = ax[p] - bx, wy = ay[p] - by;
            const double c = 3.0 * inv2 * (ux * wx + uy * wy);
            const double tx = wx - c * ux, ty = wy - c * uy;
            gx[p] += inv3 * tx;
            gy[p] += inv3 * ty;
            hx -= inv3 * tx;
            hy -= inv3 * ty;
        }
        xj = rot1d(xj);
        yj = rot1d(yj);
        bx = rot1d(bx);
        by = rot1d(by);
        hx = rot1d(hx);
        hy = rot1d(hy);
    }
}

template <int P, int W>
__global__ __launch_bounds__(64 * W) void k_adj_sym(const double4 *__restrict__ pj4, const int *__restrict__ sps,
                                                    const SymTile *__restrict__ tiles, const double *__restrict__ K,
                                                    int S, double2 *__restrict__ gpart) {
    __shared__ double2 jsum[W > 1 ? 64 * W * P : 1];
    const SymTile tl = tiles[blockIdx.x];
    const bool self = tl.j0 == tl.i0;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int ni = tl.i1 - tl.i0, nj = tl.j1 - tl.j0;
    const int a = sps[tl.i0], b = sps[tl.j0];   // a chunk holds one species
    const double kab = K[a * S + b], kba = K[b * S + a];
    double xi[P], yi[P], ax[P], ay[P], gx[P], gy[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int k = wave * 64 * P + p * 64 + lane;
        const double4 v = pj4[tl.i0 + (k < ni ? k : 0)];
        xi[p] = k < ni ? v.x : kAdjBig;
        yi[p] = k < ni ? v.y : kAdjBig;
        ax[p] = k < ni ? kab * v.z : 0.0;
        ay[p] = k < ni ? kab * v.w : 0.0;
        gx[p] = gy[p] = 0.0;
    }
    if (W > 1 && !self) {   // uniform in the workgroup
        for (int k = threadIdx.x; k < nj; k += 64 * W) jsum[k] = make_double2(0.0, 0.0);
        __syncthreads();
    }
    // wavefront w takes group (it + w * step) mod turns at turn it: no two the same at a time
    const int groups = (nj + 63) / 64;
    const int turns = groups > W ? groups : W, step = turns / W;
    for (int it = 0; it < turns; ++it) {   // same trip count in every lane
        int g = it + wave * step;
        if (g >= turns) g -= turns;
        if (g < groups) {
            const int k = g * 64 + lane;
            const double4 v = pj4[tl.j0 + (k < nj ? k : 0)];
            const double xj = k < nj ? v.x : -kAdjBig, yj = k < nj ? v.y : -kAdjBig;
            const double bx = k < nj ? kba * v.z : 0.0, by = k < nj ? kba * v.w : 0.0;
            double hx = 0.0, hy = 0.0;
            if (self)
                adj_group<P, true>(xi, yi, ax, ay, gx, gy, xj, yj, bx, by, hx, hy, g - wave * P);
            else
                adj_group<P, false>(xi, yi, ax, ay, gx, gy, xj, yj, bx, by, hx, hy, -1);
            if (!self && k < nj) {
                if (W > 1) {
                    const double2 o = jsum[k];
                    jsum[k] = make_double2(o.x + hx, o.y + hy);
                } else {
                    gpart[tl.pbase_j + tl.j0 + k] = make_double2(hx, hy);
                }
            }
        }
        if (W > 1 && !self) __syncthreads();   // the sums of this turn's groups are in place
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int k = wave * 64 * P + p * 64 + lane;
        if (k < ni) gpart[tl.pbase_i + tl.i0 + k] = make_double2(gx[p], gy[p]);
    }
    if (self || W == 1) return;   // uniform in the workgroup
    for (int k = threadIdx.x; k < nj; k += 64 * W) gpart[tl.pbase_j + tl.j0 + k] = jsum[k];
}

inline int nblocks(long long n) { return (int)((n + kAdjBlock - 1) / kAdjBlock); }

}  // namespace

// Rounds [r0, r1) of the tape, last first; dir: the host's copy of their (first entry, count).
void launch_adj_rounds(Sim &s, const int2 *dir, int r0, int r1) {
    const Tape &tp = s.adj.tape;
    AdjState &a = s.adj;
    const RoundTape t{tp.ev, tp.eold, tp.edisp, tp.ewf, tp.ecnt, tp.enb, s.rad, s.p.cap_frac, s.p.overlap_factor};
    while (r1 > r0) {
        int r = r1;
        while (r > r0 && dir[r - 1].y <= kAdjRoundMax) --r;
        if (r < r1) {
            hipLaunchKernelGGL(k_adj_rounds, dim3(1), dim3(kRoundsBlock), 0, s.stream, (const int2 *)tp.dir, r, r1, t,
                               a.lam, a.nub);
        } else {
            --r;
            const int nb = nblocks(dir[r].y);
            hipLaunchKernelGGL(k_adj_round_prep, dim3(nb), dim3(kAdjBlock), 0, s.stream, dir[r].x, dir[r].y, t,
                               (const double2 *)a.lam, a.nub);
            hipLaunchKernelGGL(k_adj_round_apply, dim3(nb), dim3(kAdjBlock), 0, s.stream, dir[r].x, dir[r].y, t,
                               (const double4 *)a.nub, a.lam);
        }
        r1 = r;
    }
}

void launch_adj_step(Sim &s, int t) {
    const Tape &tp = s.adj.tape;
    AdjState &a = s.adj;
    const int nb = nblocks(s.n);
    const double *px = tp.px + (size_t)t * s.n, *py = tp.py + (size_t)t * s.n;
    const signed char *wf = tp.emwf + (size_t)t * 2 * s.n;
    auto cast = [&](auto kern, auto *pj) {
        hipLaunchKernelGGL(kern, dim3(nb), dim3(kAdjBlock), 0, s.stream, s.n, px, py, wf, s.sorted_id, a.lam, a.pj4,
                           tp.phi ? nullptr : pj);
    };
    s.fp32 ? cast(k_adj_cast<float2>, (float2 *)s.pj) : cast(k_adj_cast<double2>, (double2 *)s.pj);
    // Phi at the positions before the step: kept by the replay, else recomputed
    const size_t vec = s.fp32 ? sizeof(float2) : sizeof(double2);
    const void *phi = tp.phi ? (const char *)tp.phi + (size_t)t * s.part_cap * vec : s.part;
    if (!tp.phi) launch_force(s, s.pj);
    if (s.persistent == 2) {   // chunk pairs, a chunk 64 W P disks
        auto go = [&](auto kern, int waves) {
            hipLaunchKernelGGL(kern, dim3(s.nstiles), dim3(64 * waves), 0, s.stream, (const double4 *)a.pj4,
                               s.sp_sorted, (const SymTile *)s.stiles, s.Kd, s.S, a.gpart);
        };
        if (s.chunk_len == 128)
            go(k_adj_sym<2, 1>, 1);
        else if (s.chunk_len == 256)
            go(k_adj_sym<4, 1>, 1);
        else if (s.chunk_len == 512)
            go(k_adj_sym<4, 2>, 2);
        else
            go(k_adj_sym<4, 4>, 4);
    } else {   // tiles of 256 min(per_lane, 4) disks
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(s.ntiles), dim3(kAdjBlock), 0, s.stream, a.pj4, s.sp_sorted, s.tiles, s.Kd,
                               s.S, a.gpart);
        };
        if (s.per_lane == 1)
            go(k_adj_pairs<1>);
        else if (s.per_lane == 2)
            go(k_adj_pairs<2>);
        else
            go(k_adj_pairs<4>);
    }
    auto update = [&](auto kern, auto *p) {
        hipLaunchKernelGGL(kern, dim3(a.dk_blocks), dim3(64 * kUpdateWaves), 0, s.stream, s.n, s.S, p,
                           (const double2 *)a.gpart, s.reps, s.rep_of, s.chunk_spec, s.sp, s.pos_of, s.p.dt, a.lam,
                           a.dk_blk);
    };
    s.fp32 ? update(k_adj_update<float2>, (const float2 *)phi) : update(k_adj_update<double2>, (const double2 *)phi);
}

void launch_adj_dk_final(Sim &s) {
    hipLaunchKernelGGL(k_adj_dk_final, dim3(s.S * s.S), dim3(kAdjBlock), 0, s.stream, s.adj.dk_blocks, s.S,
                       s.adj.dk_blk, s.adj.dk);
}

}  // namespace bd
