// Short-range forces through Verlet neighbour lists on a cell grid (Sec. 2.1
// neighbour lists with cells; Sec. 2.2 cutoff rule; Sec. 5: lists built by
// grouping the particles of each cell).
//
// Lists hold every disk j within r_list = r_cut + skin of disk i at build
// time, in a fixed order (cells of the 3 x 3 block in turn, ids ascending
// inside a cell), stored slot-major (nl[k * n + i]) for coalesced reads.
// They stay valid while no disk has moved more than skin / 2 since the build:
// then every pair with d <= r_cut at force time is in the list.  The build is
// two launches: every disk enters its cell's row, then one thread per disk scans
// the 3 x 3 rows around it, each row's few ids sorted in registers.  Cells of
// more disks than a row holds are sorted once by a launch between the two: by
// every build of the host, and in queued steps from the first such cell on (a
// step queued before halts at its force, and the host runs it again).  In graph
// mode the launches are part of every queued step and do nothing unless the
// previous step's skin test asked for new lists (`req` points at the step's
// flag; null: always build), so what they cost is their launches: as a counting
// sort (count, two scans, scatter, sort, build) six launches took 27 us of every
// step, now 9, and a build of 1,000,000 disks 166 us, now 104.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "bd_internal.h"
#include "geom.h"

namespace bd {
namespace {

// Separation component: from the nearest image in a periodic box of side P > 0, as is with walls (P = 0).
__device__ __forceinline__ double sep(double v, double P) { return P > 0.0 ? bd_min_image(v, P) : v; }
// The same with the box kind fixed at compile time: the list passes are instantiated for each kind, so
// the minimum image (an FP64 division) is absent from the wall-box kernels instead of selected per pair.
template <bool PER>
__device__ __forceinline__ double sep_k(double v, double P) { return PER ? bd_min_image(v, P) : v; }

__device__ __forceinline__ int cell_coord(double v, double inv_cell, int nc) {
    int c = (int)(v * inv_cell);
    return c < 0 ? 0 : (c >= nc ? nc - 1 : c);
}

// List passes (force, overlap gather): neighbours whose loads are issued together.
constexpr int kNlBatch = 2;

// The build kernels loop over their items with a grid of at most kBuildGrid
// workgroups: in a queued step they usually find no request and return at
// once, and a launch of few workgroups costs less.
constexpr int kBuildGrid = 512;

// A cell's row: the number of disks, then the first seven ids, in the order they came; one 32-byte sector.  Further
// disks hang on the cell's chain (cell_more: the last one + 1, cell_next: the one before, by id), and the eighth enters
// the cell in the list of long cells.  Rows and chains are empty between builds: whoever reads the new lists first
// clears them.
constexpr int kCellIds = 7;
constexpr int kCellRow = kCellIds + 1;

struct LongCells {
    int *list;   // cells of more than kCellIds disks, in the order they came
    int *ids;
    int *ctl;    // K_NL_LONG of them, K_NL_IDS of ids taken
};

__global__ void k_cell_insert(int n, const double2 *__restrict__ xy, double inv_cell, int nc, int *__restrict__ rows,
                              int *__restrict__ more, int *__restrict__ next, LongCells lc, const int *req) {
    if (req && !*req) return;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const double2 p = xy[i];
        const int c = cell_coord(p.y, inv_cell, nc) * nc + cell_coord(p.x, inv_cell, nc);
        const int k = atomicAdd(&rows[(size_t)c * kCellRow], 1);
        if (k < kCellIds) {
            rows[(size_t)c * kCellRow + 1 + k] = i;
            continue;
        }
        const unsigned long long eighth = __ballot(k == kCellIds);   // one reservation for the wavefront
        if (eighth != 0) {
            const int lane = __lane_id(), leader = __ffsll(eighth) - 1;
            int at = 0;
            if (lane == leader) at = atomicAdd(&lc.ctl[K_NL_LONG], __popcll(eighth));
            at = __shfl(at, leader);
            if (k == kCellIds) lc.list[at + __popcll(eighth & ((1ull << lane) - 1ull))] = c;
        }
        next[i] = atomicExch(&more[c], i + 1);
    }
}

// The ids of each long cell in ascending order, kSortLanes lanes a cell: gathered from the row and the chain, then each
// to the place that the number of smaller ones gives.  cell_more becomes the start of the sorted ids.  The time is the
// walk of the chain; room is taken with one atomic for all cells of a workgroup's turn (262,144 disks, 11 a cell, with
// an atomic per cell here and in the insert 399 us a build, so 151).  Unit disks at area fraction 0.5, us a build with
// every disk selecting a long cell's next id from its chain / sorted once (and as a counting sort of all cells):
// 262,144 with lists of radius 3 37 / 37 (52), 5.5 75 / 63 (90), 8.5 278 / 151 (190), 12.5 1158 / 271 (408); 40,009
// with 12.5 670 / 95 (224).
constexpr int kSortBlock = 256, kSortLanes = 8, kSortCells = kSortBlock / kSortLanes;

__global__ __launch_bounds__(kSortBlock) void k_cells_sort(const int *__restrict__ rows, int *__restrict__ more,
                                                           const int *__restrict__ next, LongCells lc,
                                                           const int *req) {
    __shared__ int start[kSortCells];
    if (req && !*req) return;
    const int g = threadIdx.x / kSortLanes, lane = threadIdx.x & (kSortLanes - 1), count = lc.ctl[K_NL_LONG];
    for (int w0 = blockIdx.x * kSortCells; w0 < count; w0 += gridDim.x * kSortCells) {   // uniform in the workgroup
        const bool valid = w0 + g < count;
        const int c = valid ? lc.list[w0 + g] : 0;
        const int *row = rows + (size_t)c * kCellRow;
        const int m = valid ? row[0] : 0;
        __syncthreads();   // the turn before has read its starts
        if (lane == 0) start[g] = 2 * m;
        __syncthreads();
        if (threadIdx.x < kSortCells) {   // one wavefront
            const int own = start[threadIdx.x];
            int incl = own;
            for (int off = 1; off < kSortCells; off <<= 1) {
                const int v = __shfl_up(incl, off, kSortCells);
                if ((int)threadIdx.x >= off) incl += v;
            }
            int at = 0;
            if (threadIdx.x == kSortCells - 1) at = atomicAdd(&lc.ctl[K_NL_IDS], incl);
            start[threadIdx.x] = __shfl(at, kSortCells - 1, kSortCells) + incl - own;
        }
        __syncthreads();
        int *came = lc.ids + start[g], *sorted = came + m;
        if (valid) {
            if (lane < kCellIds) came[lane] = row[1 + lane];
            int e = more[c];
            for (int k = kCellIds; k < m; ++k) {   // the same in the cell's lanes
                if (lane == 0) came[k] = e - 1;
                e = next[e - 1];
            }
        }
        __syncthreads();   // the ids that other lanes wrote
        for (int k = lane; k < m; k += kSortLanes) {
            const int id = came[k];
            int smaller = 0;
#pragma unroll 8
            for (int q = 0; q < m; ++q) smaller += came[q] < id ? 1 : 0;
            sorted[smaller] = id;
        }
        if (valid && lane == 0) more[c] = start[g] + m;
    }
}

// The list of disk i: neighbours within r_list from the 3 x 3 cells, in cell
// order and by id inside a cell, written straight to the slot-major list (at
// most cap; the largest count above cap is reported so the caller can grow the
// lists).  The position at build time is kept for the skin test.
struct BuildArgs {
    int n, nc, cap;
    double inv_cell, rl2, P;
    const double2 *xy;
    const int4 *rows;
    const int *more, *ids;   // ids: the sorted ids of the long cells (null: they are not sorted)
    int *nl, *nl_cnt, *overflow;
    double *xb, *yb;
};

template <bool PER>
__device__ __forceinline__ void nl_build_one(const BuildArgs &a, int i) {
#pragma clang fp contract(off)
    const double2 pi = a.xy[i];
    const int nc = a.nc;
    const int cx = cell_coord(pi.x, a.inv_cell, nc), cy = cell_coord(pi.y, a.inv_cell, nc);
    int cnt = 0;
    auto test = [&](int j, double2 pj) {
        const double dx = sep_k<PER>(pi.x - pj.x, a.P), dy = sep_k<PER>(pi.y - pj.y, a.P);
        if (j == i || dx * dx + dy * dy > a.rl2) return;
        if (cnt < a.cap) a.nl[(size_t)cnt * a.n + i] = j;
        ++cnt;
    };
    // periodic box: the 3 x 3 block wraps around (at least 3 cells a row, so no cell twice)
    for (int oy = -1; oy <= 1; ++oy) {
        int gy = cy + oy;
        if (PER)
            gy = gy < 0 ? gy + nc : (gy >= nc ? gy - nc : gy);
        else if (gy < 0 || gy >= nc)
            continue;
        int c[3];
        int4 lo[3], hi[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {   // the three rows are loaded together
            int gx = cx + u - 1;
            if (PER) gx = gx < 0 ? gx + nc : (gx >= nc ? gx - nc : gx);
            c[u] = gx < 0 || gx >= nc ? -1 : gy * nc + gx;
            const int cu = c[u] < 0 ? gy * nc + cx : c[u];
            lo[u] = a.rows[2 * (size_t)cu];
            hi[u] = a.rows[2 * (size_t)cu + 1];
        }
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const int m = c[u] < 0 ? 0 : lo[u].x;
            int id[kCellIds] = {lo[u].y, lo[u].z, lo[u].w, hi[u].x, hi[u].y, hi[u].z, hi[u].w};
            if (m > kCellIds) {
                if (!a.ids) continue;   // the step halts before its lists are read
                const int *ids = a.ids + a.more[c[u]];
                constexpr int kB = 8;
                for (int k = 0; k < m; k += kB) {
                    int j[kB];
                    double2 pj[kB];
#pragma unroll
                    for (int q = 0; q < kB; ++q) j[q] = k + q < m ? ids[k + q] : i;   // disk i is not its own neighbour
#pragma unroll
                    for (int q = 0; q < kB; ++q) pj[q] = a.xy[j[q]];
#pragma unroll
                    for (int q = 0; q < kB; ++q) test(j[q], pj[q]);
                }
                continue;
            }
#pragma unroll
            for (int q = 0; q < kCellIds; ++q)
                if (q >= m) id[q] = 0x7FFFFFFF;
#pragma unroll
            for (int r = 0; r < kCellIds; ++r)   // odd-even transposition: as many rounds as ids
#pragma unroll
                for (int q = r & 1; q + 1 < kCellIds; q += 2) {
                    const int x = id[q], y = id[q + 1];
                    id[q] = x < y ? x : y;
                    id[q + 1] = x < y ? y : x;
                }
            double2 p[kCellIds];
#pragma unroll
            for (int q = 0; q < kCellIds; ++q)
                if (q < m) p[q] = a.xy[id[q]];
#pragma unroll
            for (int q = 0; q < kCellIds; ++q)
                if (q < m) test(id[q], p[q]);
        }
    }
    if (cnt > a.cap) atomicMax(a.overflow, cnt);
    a.nl_cnt[i] = cnt < a.cap ? cnt : a.cap;
    a.xb[i] = pi.x;
    a.yb[i] = pi.y;
}

template <bool PER>
__global__ __launch_bounds__(256) void k_nl_build(BuildArgs a, const int *req) {
    if (req && !*req) return;
    for (int i = xcd_block() * blockDim.x + threadIdx.x; i < a.n; i += gridDim.x * blockDim.x) nl_build_one<PER>(a, i);
}

// Empties the cell of a disk at p (cells may be many more than disks, so by disk).
__device__ __forceinline__ void cell_clear(double2 p, double inv_cell, int nc, int *rows, int *more) {
    const int c = cell_coord(p.y, inv_cell, nc) * nc + cell_coord(p.x, inv_cell, nc);
    rows[(size_t)c * kCellRow] = 0;
    more[c] = 0;
}

__global__ void k_cells_clear(int n, const double2 *__restrict__ xy, double inv_cell, int nc, int *__restrict__ rows,
                              int *__restrict__ more) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) cell_clear(xy[i], inv_cell, nc, rows, more);
}

// Pair force over the list: F_i = sum_j K[s_i][s_j] g(d) (r_i - r_j)/d for
// d <= r_cut, g(d) = A exp(-d/lam)/d (screened) or d^-q (power).  The
// separation, its length and the cutoff test are FP64 (positions stay FP64);
// T is the precision of the law's arithmetic and of the sum (FP32 or FP64).  ONE_SPECIES: a single
// species, so no neighbour's species is read.
template <typename T, bool ONE_SPECIES, bool PER>
__global__ __launch_bounds__(256) void k_force_nl(int n, const double2 *__restrict__ xy, const int *__restrict__ sp,
                                                  const double *__restrict__ K, int S,
                                                  int kind, double q, double A, double lam, double rc,
                                                  const int *__restrict__ nl, const int *__restrict__ nl_cnt,
                                                  double2 *__restrict__ f, const StepBase *__restrict__ base,
                                                  int *__restrict__ ctl, double inv_cell, int nc,
                                                  int *__restrict__ rows, int *__restrict__ more, bool sorted,
                                                  double P) {
#pragma clang fp contract(off)
    int i = xcd_block() * blockDim.x + threadIdx.x;
    if (base->stop) return;
    // after a rebuild inside a queued step: count it, and stop the step here if a disk had more
    // neighbours than the lists hold or a cell was long and not sorted (the host grows the lists, sorts, and runs the
    // step again)
    const bool built = base->nl_now != 0;
    const bool over = built && (ctl[K_NL_OVERFLOW] > 0 || (!sorted && ctl[K_NL_LONG] > 0));
    if (built && blockIdx.x == 0 && threadIdx.x == 0) {
        ctl[K_NL_BUILT] = 1;
        if (over) {
            ctl[K_REASON] = HALT_NL_CAPACITY;
            ctl[K_STAGE] = 0;
            ctl[K_HALT] = 1;
        }
    }
    if (built && i < n) cell_clear(xy[i], inv_cell, nc, rows, more);
    if (over || i >= n) return;
    const double2 pi = xy[i];
    const double xi = pi.x, yi = pi.y;
    const int si = ONE_SPECIES ? 0 : sp[i];
    const T k0 = (T)K[0];
    const T lamT = (T)lam, AT = (T)A, qT = (T)q;
    constexpr bool F32 = sizeof(T) == 4;
    const T inv_lam = (T)(1.0 / lam);   // FP32: one reciprocal of the separation per pair instead of three divisions
    const int m = nl_cnt[i];
    T fx = (T)0, fy = (T)0;
    // kNlBatch neighbours at a time: their ids, then their positions, are all loaded before the sums,
    // which keep the list order (slots past the count read disk i itself and are not summed)
    for (int k = 0; k < m; k += kNlBatch) {
        int jb[kNlBatch];
#pragma unroll
        for (int u = 0; u < kNlBatch; ++u) jb[u] = k + u < m ? nl[(size_t)(k + u) * n + i] : i;
        double xj[kNlBatch], yj[kNlBatch];
        int sj[kNlBatch];
#pragma unroll
        for (int u = 0; u < kNlBatch; ++u) {
            const double2 pj = xy[jb[u]];
            xj[u] = pj.x;
            yj[u] = pj.y;
            sj[u] = ONE_SPECIES ? 0 : sp[jb[u]];
        }
#pragma unroll
        for (int u = 0; u < kNlBatch; ++u) {
            if (k + u >= m) break;
            const double ddx = sep_k<PER>(xi - xj[u], P), ddy = sep_k<PER>(yi - yj[u], P);
            const double dd = sqrt(ddx * ddx + ddy * ddy);
            if (dd > rc) continue;   // the cutoff decision in FP64 in both precisions
            const T dx = (T)ddx, dy = (T)ddy, d = (T)dd;
            T s;
            if (kind == BD_FORCE_SCREENED) {
                if (F32) {
                    const T r = (T)1 / d;
                    s = AT * exp(-d * inv_lam) * (r * r);
                } else {
                    s = AT * exp(-d / lamT) / d / d;
                }
            } else
                s = pow(d, -qT) / d;
            s *= ONE_SPECIES ? k0 : (T)K[si * S + sj[u]];
            fx += s * dx;
            fy += s * dy;
        }
    }
    f[i] = make_double2((double)fx, (double)fy);
}

// Skin test at the end of a step: has any disk moved more than skin / 2 since
// the lists were built?  (strict, displacement including corrections and walls)
// The request also goes to the step base, where the next queued step finds it.
// (Steps queued after one that halted run it too, harmlessly: the host clears
// both flags before it tests the halted step's final positions itself.)
__global__ void k_skin_check(int n, const double *__restrict__ x, const double *__restrict__ y,
                             const double *__restrict__ xb, const double *__restrict__ yb, double half_skin2,
                             int *__restrict__ flag, StepBase *__restrict__ base, double P) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    bool out = false;
    if (i < n) {
        const double dx = sep(x[i] - xb[i], P), dy = sep(y[i] - yb[i], P);
        out = dx * dx + dy * dy > half_skin2;
    }
    if (__ballot(out) != 0 && __lane_id() == 0) {
        atomicOr(flag, 1);
        atomicOr(&base->nl_req, 1);
    }
}

// ---------------------------------------------------------------- overlap rounds over the lists
// The paper's short-range variant (Sec. 5) finds overlapping pairs through the
// neighbour lists instead of a triangulation.  Round k, gather: every disk sums
// its Jacobi displacement over the listed partners that overlap it (Sec. 2.3
// displacement along the unit vector, factor f), truncates the sum to
// cap_frac * r (Sec. 4.4) and applies the walls; a disk that moved is queued
// with its new position.  Overlapping pairs are counted once (from the lower
// id).  The lists contain every pair closer than contact only while no disk
// has moved more than `margin` since the build; a disk beyond it raises
// K_NL_STALE and the round is not applied (the host rebuilds the lists and
// repeats the detection).  Apply: if the round found nothing the overlap loop
// is done; otherwise the queued disks take their new positions (all at once,
// after every gather has read the old ones).
// Workgroups of 1024 threads, at most kNlGatherGrid of them, each disk once
// (grid-stride): the disks a workgroup queues are staged in LDS with their
// new positions and reserved on the shared counter once per workgroup, and the
// pair, cap and stale counts are added once per workgroup (updates of one
// address from every CU serialise).
constexpr int kNlGatherBlock = 1024;
constexpr int kNlGatherGrid = 512;
constexpr int kNlStage = 2048;

// UNI: every disk has the same radius (the contact distance is then 2 r_i, the same value rad[i] + rad[j]
// gives), so the neighbours' radii are not loaded.
// The arguments of the overlap rounds over the lists.
struct NlArgs {
    int n;
    const double2 *xy;
    const double *rad;
    double L;
    const int *nl, *nl_cnt;
    const double *xb, *yb;
    double margin2, f, cap_frac, keep, P;
};

// Round k's gather for disk i: the sum over its listed neighbours closer than
// contact (in list order), truncated to cap_frac * r_i, walls or wrap; moved
// when it has an overlapping neighbour.  Counts the overlapping pairs it owns
// (the lower id), cap hits, and whether the disk is beyond the list margin.
template <bool PER, bool UNI>
__device__ __forceinline__ void nl_gather_disk(const NlArgs &a, int i, bool &moved, double &nx, double &ny,
                                               int &pairs, int &caps, bool &stale_any) {
#pragma clang fp contract(off)
    const int n = a.n;
    const double2 *__restrict__ xy = a.xy;
    const double *__restrict__ rad = a.rad;
    const int *__restrict__ nl = a.nl;
    const double P = a.P, keep = a.keep, f = a.f;
    const double2 pi = xy[i];
    const double xi = pi.x, yi = pi.y, ri = rad[i];
    const double ex = sep_k<PER>(xi - a.xb[i], P), ey = sep_k<PER>(yi - a.yb[i], P);
    stale_any |= ex * ex + ey * ey > a.margin2;
    const int m = a.nl_cnt[i];
    double sx = 0.0, sy = 0.0;
    for (int q = 0; q < m; q += kNlBatch) {   // batched loads as in k_force_nl, sums in list order
        int jb[kNlBatch];
#pragma unroll
        for (int u = 0; u < kNlBatch; ++u) jb[u] = q + u < m ? nl[(size_t)(q + u) * n + i] : i;
        double xj[kNlBatch], yj[kNlBatch], rj[kNlBatch];
#pragma unroll
        for (int u = 0; u < kNlBatch; ++u) {
            const double2 pj = xy[jb[u]];
            xj[u] = pj.x;
            yj[u] = pj.y;
            rj[u] = UNI ? ri : rad[jb[u]];
        }
#pragma unroll
        for (int u = 0; u < kNlBatch; ++u) {
            if (q + u >= m) break;
            const double dx = sep_k<PER>(xi - xj[u], P), dy = sep_k<PER>(yi - yj[u], P);
            const double d = sqrt(dx * dx + dy * dy);
            const double contact = ri + rj[u];
            if (d < contact * keep) {
                const double sc = f * (contact - d) / d;
                sx += sc * dx;
                sy += sc * dy;
                moved = true;
                if (i < jb[u]) ++pairs;
            }
        }
    }
    if (moved) {
        const double len = sqrt(sx * sx + sy * sy);
        const double cap = a.cap_frac * ri;
        if (len > cap) {
            const double sc = cap / len;
            sx = sx * sc;
            sy = sy * sc;
            ++caps;
        }
        nx = PER ? bd_wrap(xi + sx, P) : bd_wall(xi + sx, ri, a.L);
        ny = PER ? bd_wrap(yi + sy, P) : bd_wall(yi + sy, ri, a.L);
    }
}

template <bool PER, bool UNI>
__global__ __launch_bounds__(kNlGatherBlock) void k_ovl_nl_gather(NlArgs a, int *__restrict__ touched,
                                                                  double2 *__restrict__ newpos, int *__restrict__ ctl,
                                                                  unsigned long long *__restrict__ acc, int k) {
#pragma clang fp contract(off)
    const int n = a.n;
    __shared__ int s_id[kNlStage];
    __shared__ double2 s_pos[kNlStage];
    __shared__ int s_cnt, s_base, s_pairs, s_caps, s_stale;
    if ((ctl[K_HALT] | ctl[K_DONE]) != 0) return;   // nothing in this launch writes them: uniform
    if (threadIdx.x == 0) {
        s_cnt = 0;
        s_pairs = 0;
        s_caps = 0;
        s_stale = 0;
    }
    __syncthreads();
    int pairs = 0, caps = 0;
    bool stale_any = false;
    const int stride = gridDim.x * blockDim.x;
    for (int i0 = xcd_block() * blockDim.x; i0 < n; i0 += stride) {   // same trip count in the workgroup
        const int i = i0 + (int)threadIdx.x;
        bool moved = false;
        double nx = 0.0, ny = 0.0;
        if (i < n) nl_gather_disk<PER, UNI>(a, i, moved, nx, ny, pairs, caps, stale_any);
        // stage the queued disk (one LDS atomic per wavefront; every lane is here)
        const unsigned long long mm = __ballot(moved);
        if (mm != 0) {
            const int lane = __lane_id(), leader = __ffsll((unsigned long long)mm) - 1;
            int base = 0;
            if (lane == leader) base = atomicAdd(&s_cnt, __popcll(mm));
            base = __shfl(base, leader);
            if (moved) {
                const int pos = base + __popcll(mm & ((1ull << lane) - 1ull));
                if (pos < kNlStage) {
                    s_id[pos] = i;
                    s_pos[pos] = make_double2(nx, ny);
                } else {
                    const int g = atomicAdd(&ctl[K_TOUCH + k], 1);
                    touched[g] = i;
                    newpos[g] = make_double2(nx, ny);
                }
            }
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        pairs += __shfl_xor(pairs, off);
        caps += __shfl_xor(caps, off);
    }
    const bool stale_w = __ballot(stale_any) != 0;
    if (__lane_id() == 0) {
        if (pairs) atomicAdd(&s_pairs, pairs);
        if (caps) atomicAdd(&s_caps, caps);
        if (stale_w) s_stale = 1;
    }
    __syncthreads();
    const int cnt = s_cnt < kNlStage ? s_cnt : kNlStage;
    if (threadIdx.x == 0) {
        if (cnt > 0) s_base = atomicAdd(&ctl[K_TOUCH + k], cnt);
        if (s_pairs) atomicAdd(&ctl[K_OVL + k], s_pairs);
        if (s_caps) atomicAdd(&acc[A_CAP_HITS], (unsigned long long)s_caps);
        if (s_stale) atomicOr(&ctl[K_NL_STALE], 1);
    }
    __syncthreads();
    for (int q = threadIdx.x; q < cnt; q += blockDim.x) {
        touched[s_base + q] = s_id[q];
        newpos[s_base + q] = s_pos[q];
    }
}

// final_check: the last budgeted round's detection; overlaps left halt the
// step (the host continues the loop) instead of being applied.
__global__ __launch_bounds__(256) void k_ovl_nl_apply(double *__restrict__ x, double *__restrict__ y,
                                                      double2 *__restrict__ xy,
                                                      const int *__restrict__ touched,
                                                      const double2 *__restrict__ newpos, int *__restrict__ ctl, int k,
                                                      int final_check) {
    if ((ctl[K_HALT] | ctl[K_DONE]) != 0) return;
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    // the counters below were written by the gather launch before this one: every thread reads the same
    if (ctl[K_NL_STALE] != 0) {
        if (lead) {
            ctl[K_REASON] = HALT_NL_STALE;
            ctl[K_STAGE] = k;
            ctl[K_HALT] = 1;
        }
        return;
    }
    if (ctl[K_OVL + k] == 0) {
        if (lead) ctl[K_DONE] = 1;
        return;
    }
    if (final_check) {
        if (lead) {
            ctl[K_REASON] = HALT_OVERLAP_BUDGET;
            ctl[K_STAGE] = k;
            ctl[K_HALT] = 1;
        }
        return;
    }
    if (lead) ctl[K_OVL_ROUNDS] = k + 1;
    const int cnt = ctl[K_TOUCH + k];
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < cnt; idx += gridDim.x * blockDim.x) {
        const int v = touched[idx];
        const double2 p = newpos[idx];
        x[v] = p.x;
        y[v] = p.y;
        xy[v] = p;
    }
}

// The later overlap rounds over the lists in one workgroup.  After a round,
// only a disk that moved in it, or a listed neighbour of one, can overlap
// another (a pair whose disks both stayed keeps its distance, and every disk
// that had an overlapping neighbour moved): round r gathers over exactly those
// disks (each once, marked with the round's stamp), with the arithmetic of the
// full pass, so it moves the same disks to the same places and counts the same
// pairs; the margin test of a disk that did not move since its last test would
// give the same answer.  Each round ends as k_ovl_nl_apply does (lists stale:
// halt; no overlap: done; the budget's last round with overlaps left: halt;
// else the queued disks take their positions), phases separated by barriers.
constexpr int kNlTailBlock = 1024;

__device__ __forceinline__ bool nl_stopped(const int *ctl) {
    return (__hip_atomic_load(ctl + K_HALT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) |
            __hip_atomic_load(ctl + K_DONE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0;
}

// (xyw is the array a.xy reads: the gathers and the position writes of a round are separated by barriers.)
template <bool PER, bool UNI>
__global__ __launch_bounds__(kNlTailBlock) void k_nl_tail(NlArgs a, NlTailPlan p, double *x, double *y, double2 *xyw,
                                                          int *touched, double2 *newpos, int *mark, int *cand,
                                                          int *ctl, unsigned long long *acc,
                                                          const StepBase *__restrict__ base) {
    __shared__ int s_nc, s_cnt, s_pairs, s_caps, s_stale, s_go;
    const int tid = threadIdx.x, n = a.n;
    // the decisions every thread follows are taken by thread 0 and read from LDS after a barrier
    if (tid == 0) s_go = nl_stopped(ctl) ? 0 : 1;
    __syncthreads();
    if (!s_go) return;
    int kprev = p.kprev;
    for (int r = 0; r < p.nr; ++r) {
        const int k = p.k[r];
        const int stamp = p.stamp0 + r + base->vbase;
        if (tid == 0) {
            s_nc = 0;
            s_cnt = 0;
            s_pairs = 0;
            s_caps = 0;
            s_stale = 0;
        }
        __syncthreads();
        // the disks of this round: those the previous round moved and their listed neighbours
        const int nprev = ctl[K_TOUCH + kprev];
        const int *prev = touched + (size_t)(kprev & 1) * n;
        for (int idx = tid; idx < nprev; idx += kNlTailBlock) {
            const int v = prev[idx];
            if ((unsigned)v >= (unsigned)n) continue;
            if (atomicExch(&mark[v], stamp) != stamp) cand[atomicAdd(&s_nc, 1)] = v;
            const int m = a.nl_cnt[v];
            for (int q = 0; q < m; ++q) {
                const int w = a.nl[(size_t)q * n + v];
                if (atomicExch(&mark[w], stamp) != stamp) cand[atomicAdd(&s_nc, 1)] = w;
            }
        }
        __syncthreads();
        const int nc = s_nc;
        int *cur = touched + (size_t)(k & 1) * n;
        int pairs = 0, caps = 0;
        bool stale = false;
        for (int c = tid; c < nc; c += kNlTailBlock) {
            const int i = cand[c];
            bool moved = false;
            double nx = 0.0, ny = 0.0;
            nl_gather_disk<PER, UNI>(a, i, moved, nx, ny, pairs, caps, stale);
            if (moved) {
                const int g = atomicAdd(&s_cnt, 1);
                cur[g] = i;
                newpos[g] = make_double2(nx, ny);
            }
        }
        for (int off = 32; off > 0; off >>= 1) {
            pairs += __shfl_xor(pairs, off);
            caps += __shfl_xor(caps, off);
        }
        const bool stale_w = __ballot(stale) != 0;
        if (__lane_id() == 0) {
            if (pairs) atomicAdd(&s_pairs, pairs);
            if (caps) atomicAdd(&s_caps, caps);
            if (stale_w) s_stale = 1;
        }
        __syncthreads();
        if (tid == 0) {
            ctl[K_TOUCH + k] = s_cnt;
            ctl[K_OVL + k] += s_pairs;
            if (s_caps) atomicAdd(&acc[A_CAP_HITS], (unsigned long long)s_caps);
            if (s_stale) {
                ctl[K_NL_STALE] = 1;
                ctl[K_REASON] = HALT_NL_STALE;
                ctl[K_STAGE] = k;
                ctl[K_HALT] = 1;
            } else if (s_pairs == 0) {
                ctl[K_DONE] = 1;
            } else if (p.final_last && r + 1 == p.nr) {
                ctl[K_REASON] = HALT_OVERLAP_BUDGET;
                ctl[K_STAGE] = k;
                ctl[K_HALT] = 1;
            } else {
                ctl[K_OVL_ROUNDS] = k + 1;
            }
            s_go = ctl[K_HALT] == 0 && ctl[K_DONE] == 0;
        }
        __syncthreads();
        if (!s_go) return;
        const int cnt = s_cnt;
        for (int idx = tid; idx < cnt; idx += kNlTailBlock) {
            const int v = cur[idx];
            const double2 np = newpos[idx];
            x[v] = np.x;
            y[v] = np.y;
            xyw[v] = np;
        }
        __syncthreads();
        kprev = k;
    }
}

inline int blocks(int n) { return (n + 255) / 256; }
inline int capped(int b, int cap = kBuildGrid) { return b < 1 ? 1 : (b > cap ? cap : b); }

NlArgs nl_args(const Sim &s) {
    NlArgs a;
    a.n = s.n;
    a.xy = s.xy;
    a.rad = s.rad;
    a.L = s.L_h[0];
    a.nl = s.nl;
    a.nl_cnt = s.nl_cnt;
    a.xb = s.xbuild;
    a.yb = s.ybuild;
    a.margin2 = s.nl_margin * s.nl_margin;
    a.f = s.p.overlap_factor;
    a.cap_frac = s.p.cap_frac;
    a.keep = 1.0 - s.p.contact_tol;
    a.P = s.period;
    return a;
}

}  // namespace

namespace {

// The build kernels; req = null builds unconditionally, else only when *req != 0.
void enqueue_build(Sim &s, const int *req, bool sort) {
    const double rl = s.fp.cutoff + s.fp.skin;
    BuildArgs a;
    a.n = s.n;
    a.nc = s.nl_nc;
    a.cap = s.nl_cap;
    a.inv_cell = (double)s.nl_nc / s.L_h[0];
    a.rl2 = rl * rl;
    a.P = s.period;
    a.xy = s.xy;
    a.rows = (const int4 *)s.cell_rows;
    a.more = s.cell_more;
    a.ids = sort ? s.cell_ids : nullptr;
    a.nl = s.nl;
    a.nl_cnt = s.nl_cnt;
    a.overflow = s.ctl + K_NL_OVERFLOW;
    a.xb = s.xbuild;
    a.yb = s.ybuild;
    const LongCells lc{s.cell_long, s.cell_ids, s.ctl};
    hipLaunchKernelGGL(k_cell_insert, dim3(capped(blocks(s.n))), dim3(256), 0, s.stream, s.n, a.xy, a.inv_cell, a.nc,
                       s.cell_rows, s.cell_more, s.cell_next, lc, req);
    if (sort)
        hipLaunchKernelGGL(k_cells_sort, dim3(capped(s.n / 8 / kSortCells + 1, 2 * kBuildGrid)), dim3(kSortBlock), 0,
                           s.stream, (const int *)s.cell_rows, s.cell_more, (const int *)s.cell_next, lc, req);
    hipLaunchKernelGGL(s.period > 0.0 ? k_nl_build<true> : k_nl_build<false>, dim3(capped(blocks(s.n), 2 * kBuildGrid)),
                       dim3(256), 0, s.stream, a, req);
}

}  // namespace

// Ints in the rows of ncell cells.
size_t verlet_row_ints(int ncell) { return (size_t)ncell * kCellRow; }

static void launch_cells_clear(Sim &s) {
    hipLaunchKernelGGL(k_cells_clear, dim3(blocks(s.n)), dim3(256), 0, s.stream, s.n, (const double2 *)s.xy,
                       (double)s.nl_nc / s.L_h[0], s.nl_nc, s.cell_rows, s.cell_more);
}

// Rebuilds the lists from the current positions (the caller zeroed the build's counters) and empties the cells.
void launch_verlet_build(Sim &s) {
    enqueue_build(s, nullptr, true);
    launch_cells_clear(s);
}

void launch_verlet_build_requested(Sim &s) {
    StepBase *b = (StepBase *)s.dbase;
    // the force kernel that follows records the rebuild, checks its capacity and empties the cells
    enqueue_build(s, &b->nl_now, s.nl_sort);
}

void launch_force_nl(Sim &s) {
    const bool per = s.period > 0.0;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(blocks(s.n)), dim3(256), 0, s.stream, s.n, (const double2 *)s.xy,
                           (const int *)s.sp, (const double *)s.Kd, s.S, s.fp.kind, s.fp.q,
                           s.fp.A, s.fp.lambda, s.fp.cutoff, (const int *)s.nl, (const int *)s.nl_cnt, s.fsr,
                           (const StepBase *)s.dbase, s.ctl, (double)s.nl_nc / s.L_h[0], s.nl_nc, s.cell_rows,
                           s.cell_more, s.nl_sort, s.period);
    };
    if (s.fp32)
        per ? (s.S == 1 ? go(k_force_nl<float, true, true>) : go(k_force_nl<float, false, true>))
            : (s.S == 1 ? go(k_force_nl<float, true, false>) : go(k_force_nl<float, false, false>));
    else
        per ? (s.S == 1 ? go(k_force_nl<double, true, true>) : go(k_force_nl<double, false, true>))
            : (s.S == 1 ? go(k_force_nl<double, true, false>) : go(k_force_nl<double, false, false>));
}

void launch_ovl_nl_gather(Sim &s, int k) {
    const int g = std::max(1, std::min(kNlGatherGrid, (s.n + kNlGatherBlock - 1) / kNlGatherBlock));
    const bool per = s.period > 0.0, uni = s.rad_uni > 0.0;
    hipLaunchKernelGGL(per ? (uni ? k_ovl_nl_gather<true, true> : k_ovl_nl_gather<true, false>)
                           : (uni ? k_ovl_nl_gather<false, true> : k_ovl_nl_gather<false, false>),
                       dim3(g), dim3(kNlGatherBlock), 0, s.stream, nl_args(s), s.touched + (size_t)(k & 1) * s.n,
                       s.newpos, s.ctl, s.acc, k);
}

void launch_nl_tail(Sim &s, const NlTailPlan &p) {
    const bool per = s.period > 0.0, uni = s.rad_uni > 0.0;
    hipLaunchKernelGGL(per ? (uni ? k_nl_tail<true, true> : k_nl_tail<true, false>)
                           : (uni ? k_nl_tail<false, true> : k_nl_tail<false, false>),
                       dim3(1), dim3(kNlTailBlock), 0, s.stream, nl_args(s), p, s.x, s.y, s.xy, s.touched, s.newpos,
                       s.vstamp, s.nl_cand, s.ctl, s.acc, (const StepBase *)s.dbase);
}

void launch_ovl_nl_apply(Sim &s, int k, bool final_check) {
    // the queued disks are usually a few percent of all: a grid for a tenth of them
    const int g = std::max(1, std::min(blocks(s.n), blocks(s.n / 10 + 1)));
    hipLaunchKernelGGL(k_ovl_nl_apply, dim3(g), dim3(256), 0, s.stream, s.x, s.y, s.xy,
                       (const int *)(s.touched + (size_t)(k & 1) * s.n), (const double2 *)s.newpos, s.ctl, k,
                       final_check ? 1 : 0);
}

void launch_skin_check(Sim &s) {
    const double h = 0.5 * s.fp.skin;
    hipLaunchKernelGGL(k_skin_check, dim3(blocks(s.n)), dim3(256), 0, s.stream, s.n, s.x, s.y, s.xbuild, s.ybuild,
                       h * h, s.ctl + K_NL_REBUILD, (StepBase *)s.dbase, s.period);
}

}  // namespace bd
