// Device-resident Delaunay triangulation: parallel edge-flip repair (Sec. 4.1
// and 4.3) and overlap correction over Delaunay edges (Sec. 2.3, 4.4,
// Algorithm 2).
//
// Triangulation layout (SoA, ghosts included).  A handle holds R independent
// systems (R = 1 for one system).  Vertex ids: the disks of all systems
// (0..n-1, system by system), their fixed frame points outside the walls
// (n..nv-1), then one infinite vertex per system (nv..nv+R-1); system r has
// 2 nv_r - 2 triangles and no edge between two systems.
//   he_v[h]     origin vertex of half-edge h; triangle t owns h = 3t..3t+2 CCW
//   he_twin[h]  opposite half-edge
//   vert_he[v]  one outgoing half-edge of vertex v
//
// One flip round is three launches:
//   eval   every candidate edge (all edges, or a worklist) applies the flip
//          rule; a flipping edge claims both of its triangles with a 64-bit
//          atomicMax of (round << 32 | ~edge): the newest round wins over stale
//          claims and, inside a round, the lowest edge id wins, independent of
//          scheduling.
//   apply  an edge that holds both claims rewrites its two triangles in place,
//          records where its four outer half-edges moved and stamps the two
//          triangles with the round.
//   fix    each flipped quad repairs the twin links of its outer half-edges
//          (through `moved` when the neighbour flipped in the same round) and
//          queues the edges whose status may have changed to the next
//          worklist; a candidate that lost without any neighbour flipping
//          re-queues itself.
// The globally lowest candidate always wins both claims, so every round with a
// candidate makes progress.
//
// Control.  Work counts live in the device control block `ctl` in per-round
// and per-overlap-round slots, so a whole step can be enqueued without the
// host reading anything back: every kernel reads its count from `ctl` and
// returns at once when the step has halted (an error or an exhausted budget,
// left for the host to finish) or the overlap loop is done.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "bd_internal.h"
#include "geom.h"
#include "step_end.h"

namespace bd {
namespace {

constexpr int kMaxGrid = 512;      // full scans over triangles that take per-workgroup atomics
constexpr int kScanGrid = 4096;    // full scans without them (many waves in flight hide the gathers' latency)
constexpr int kScanBlock = 1024;   // full scans with per-workgroup atomics: few workgroups, many waves
constexpr int kStarGridMax = 1024;  // launches with one group of lanes per star
constexpr int kListGridMax = 256;  // worklist-driven launches (usually a few hundred items, often none)

struct Topo {
    int n, inf, nvert, T;   // disks, first infinite-vertex id, all vertex ids, triangles
    double P;               // > 0: periodic box of this side (torus triangulation, minimum-image geometry)
    double ru;              // > 0: every disk has this radius (a contact distance is 2 ru, radii are not loaded)
    const int *rep_of;      // replica of each disk
    const double *Lr;       // box side of each replica
    const double *x, *y, *xo, *yo, *rad;
    const double2 *xy;      // (x, y) pairs, kept equal to x, y: the gathers of other vertices' positions load these
    int *he_v, *he_twin, *vert_he;
    unsigned long long *claim;
    int *tri_stamp, *moved, *edge_stamp, *vstamp;
    int2 *cand;
    int *cand_won;
    int *wl0, *wl1;
    int *touched;           // [2][n], by overlap-round parity
    int *det_stamp, *fl_stamp, *fl, *vt_stamp, *vt;
    double2 *newpos, *oldpos;
    int *star, *star_deg;   // star of each queued disk as its round's gather found it (see star_walk)
    int *ctl;
    unsigned long long *acc;
    const StepBase *base;   // stamps passed to kernels are relative to base->rbase / base->vbase
    // adjoint tape (null unless a segment is being recorded)
    int *tev, *tecnt, *tenb;
    double2 *teold, *tedisp;
    signed char *tewf;
    int2 *tdir;
    int tent_base, tdir_base, tcap_ent, tcap_dir;
};

Topo topo_of(Sim &s) {
    Topo t;
    t.n = s.n;
    t.inf = s.inf;
    t.P = s.period;
    t.ru = s.rad_uni;
    t.nvert = s.inf + s.R;
    t.rep_of = s.rep_of;
    t.Lr = s.Lr;
    t.T = s.T;
    t.x = s.x;
    t.y = s.y;
    t.xy = s.xy;
    t.xo = s.xo;
    t.yo = s.yo;
    t.rad = s.rad;
    t.he_v = s.he_v;
    t.he_twin = s.he_twin;
    t.vert_he = s.vert_he;
    t.claim = s.claim;
    t.tri_stamp = s.tri_stamp;
    t.moved = s.moved;
    t.edge_stamp = s.edge_stamp;
    t.vstamp = s.vstamp;
    t.cand = s.cand;
    t.cand_won = s.cand_won;
    t.wl0 = s.wl[0];
    t.wl1 = s.wl[1];
    t.touched = s.touched;
    t.det_stamp = s.det_stamp;
    t.fl_stamp = s.fl_stamp;
    t.fl = s.fl;
    t.vt_stamp = s.vt_stamp;
    t.vt = s.vt;
    t.newpos = s.newpos;
    t.oldpos = s.oldpos;
    t.star = s.star;
    t.star_deg = s.star_deg;
    t.ctl = s.ctl;
    t.acc = s.acc;
    t.base = s.dbase;
    const Tape &tp = s.adj.tape;
    const bool rec = tp.on;
    t.tev = rec ? tp.ev : nullptr;
    t.tecnt = tp.ecnt;
    t.tenb = tp.enb;
    t.teold = tp.eold;
    t.tedisp = tp.edisp;
    t.tewf = tp.ewf;
    t.tdir = tp.dir;
    t.tent_base = tp.ent_base;
    t.tdir_base = tp.dir_base;
    t.tcap_ent = tp.cap_ent;
    t.tcap_dir = tp.cap_dir;
    return t;
}

// The box kind at compile time: the kernels that read geometry are instantiated for walls and for the periodic
// box, so that the wall-box code holds no minimum images (an FP64 division each).  A kernel's code is read through a
// cache of 64 KiB shared by two compute units, and a one-workgroup kernel that walks through more than that waits
// for its instructions.
template <bool PER>
struct TopoP : Topo {
    static constexpr bool kPer = PER;
};

__device__ __forceinline__ bool stopped(const int *ctl) { return (ctl[K_HALT] | ctl[K_DONE]) != 0; }
// Read of a counter that other workgroups of the running launch update with atomics.
__device__ __forceinline__ int ctl_read(const int *ctl, int i) {
    return __hip_atomic_load(ctl + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Disks queued by overlap round k (two buffers, so a round can read the previous round's list).
__device__ __forceinline__ int *touched_of(const Topo &t, int k) { return t.touched + (size_t)(k & 1) * t.n; }
__device__ __forceinline__ int *wl_of(const Topo &t, int slot) { return (slot & 1) ? t.wl1 : t.wl0; }

// Range guards: a corrupt triangulation must never turn into an out-of-bounds
// access; it is reported through K_TOPO and repaired on the host.
__device__ __forceinline__ bool bad_he(const Topo &t, int h) { return (unsigned)h >= (unsigned)(3 * t.T); }
__device__ __forceinline__ bool bad_v(const Topo &t, int v) { return (unsigned)v >= (unsigned)t.nvert; }
__device__ __forceinline__ void topo_err(const Topo &t) { atomicAdd(&t.ctl[K_TOPO], 1); }

// Geometry of the triangulation.  With walls the vertex positions are used as
// they are.  In a periodic box (P > 0) a triangle or a quad is read in the
// frame of its first vertex, every other vertex at its nearest image: every
// edge of the torus triangulation is far shorter than P / 2, so that image is
// the one the triangle spans.
template <class TP>
__device__ __forceinline__ double sep_p(const TP &t, double v) { return TP::kPer ? bd_min_image(v, t.P) : v; }

template <class TP>
__device__ __forceinline__ int flip_rule_at(const TP &t, int a, int b, int c, int d, double2 pa, double2 pb,
                                            double2 pc, double2 pd, bool *inverted) {
    if (!TP::kPer)
        return bd_flip_rule_xy(a, b, c, d, t.inf, pa.x, pa.y, pb.x, pb.y, pc.x, pc.y, pd.x, pd.y, true, inverted);
    return bd_flip_rule_quad(0.0, 0.0, sep_p(t, pb.x - pa.x), sep_p(t, pb.y - pa.y), sep_p(t, pc.x - pa.x),
                             sep_p(t, pc.y - pa.y), sep_p(t, pd.x - pa.x), sep_p(t, pd.y - pa.y), true, inverted);
}

template <class TP>
__device__ __forceinline__ double orient_at(const TP &t, double2 pa, double2 pb, double2 pc) {
    if (!TP::kPer) return bd_orient(pa.x, pa.y, pb.x, pb.y, pc.x, pc.y);
    return bd_orient(0.0, 0.0, sep_p(t, pb.x - pa.x), sep_p(t, pb.y - pa.y), sep_p(t, pc.x - pa.x),
                     sep_p(t, pc.y - pa.y));
}

__device__ __forceinline__ unsigned long long claim_key(int round, int e) {
    return ((unsigned long long)(unsigned)round << 32) | (unsigned long long)(0xFFFFFFFFu - (unsigned)e);
}

// Counters shared by the whole grid are updated once per wavefront: lanes
// that take a list position get consecutive ones from a single atomic, and
// event counts are summed over the wavefront first (same-address atomics
// serialise in the cache, and thousands of them per launch dominate a scan).
__device__ __forceinline__ int wave_reserve(int *counter, bool want) {
    const unsigned long long m = __ballot(want);
    if (m == 0) return -1;
    const int lane = __lane_id();
    const int leader = __ffsll((unsigned long long)m) - 1;
    int base = 0;
    if (lane == leader) base = atomicAdd(counter, __popcll(m));
    base = __shfl(base, leader);
    return want ? base + __popcll(m & ((1ull << lane) - 1ull)) : -1;
}

// Sum over the (fully active) wavefront, added by one lane.
__device__ __forceinline__ void wave_sum_add(int *counter, int v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if (__lane_id() == 0 && v != 0) atomicAdd(counter, v);
}

__device__ __forceinline__ void wave_count(int *counter, bool event) {
    const unsigned long long m = __ballot(event);
    if (m != 0 && __lane_id() == __ffsll((unsigned long long)m) - 1) atomicAdd(counter, __popcll(m));
}

__device__ __forceinline__ void wave_count64(unsigned long long *counter, bool event) {
    const unsigned long long m = __ballot(event);
    if (m != 0 && __lane_id() == __ffsll((unsigned long long)m) - 1)
        atomicAdd(counter, (unsigned long long)__popcll(m));
}

// Whether the calling workgroup is the last of the grid to get here; every
// thread of every workgroup calls it once, at the end of the kernel, thread 0
// with released = true if it added to a counter the check reads.  The last
// one sees those counters complete (each adder releases before its ticket,
// the last taker acquires after) and resets the ticket for the next launch.
// An index error (K_TOPO) may reach the check late; the host reads it at the
// end of the step.  A check
// that would otherwise be a one-thread launch of its own runs there.
__device__ __forceinline__ bool last_workgroup(int *ctl, bool released) {
    __shared__ int last;
    // the counters a check reads are added by thread 0 of each workgroup: it
    // releases them before the ticket is taken (no acquire here, which would
    // drop the cache for the wavefronts still running)
    if (released) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __syncthreads();
    if (threadIdx.x == 0) {
        last = atomicAdd(&ctl[K_TICKET], 1) == (int)gridDim.x - 1;
        if (last) {
            atomicExch(&ctl[K_TICKET], 0);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
    }
    __syncthreads();
    return last != 0;
}

// Workgroup staging of worklist appends (LDS): lanes take stage positions
// with one LDS atomic per wavefront; at the end of the launch the workgroup
// reserves its entries on the shared counter with one atomic and copies them
// out.  Entries beyond the stage's capacity go to the list directly.
template <int CAP>
struct Stage {
    int buf[CAP];
    int cnt, base;
};

template <int CAP>
__device__ __forceinline__ void stage_init(Stage<CAP> &st) {
    if (threadIdx.x == 0) st.cnt = 0;
    __syncthreads();
}

// Every thread of the workgroup calls it once, at the end.
template <int CAP>
__device__ __forceinline__ void stage_flush(Stage<CAP> &st, int *counter, int *list) {
    __syncthreads();
    const int n = st.cnt < CAP ? st.cnt : CAP;
    if (threadIdx.x == 0 && n > 0) st.base = atomicAdd(counter, n);
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) list[st.base + i] = st.buf[i];
}

// Appends edge e to the worklist of round slot `slot` once per stamp.  The
// lanes of a wavefront that push at the same time take their positions with
// one atomic, on the workgroup's stage when there is one, else on the shared
// counter.
template <int CAP = 1>
__device__ __forceinline__ void push_edge(const Topo &t, int e, int stamp, int slot, Stage<CAP> *st = nullptr) {
    const bool fresh = atomicExch(&t.edge_stamp[e], stamp) != stamp;
    const unsigned long long m = __ballot(fresh);
    if (m == 0) return;
    const int lane = __lane_id();
    const int leader = __ffsll((unsigned long long)m) - 1;
    int base = 0;
    if (lane == leader) base = atomicAdd(st ? &st->cnt : &t.ctl[K_WL + slot], __popcll(m));
    base = __shfl(base, leader);
    if (!fresh) return;
    const int pos = base + __popcll(m & ((1ull << lane) - 1ull));
    if (!st)
        wl_of(t, slot)[pos] = e;
    else if (pos < CAP)
        st->buf[pos] = e;
    else
        wl_of(t, slot)[atomicAdd(&t.ctl[K_WL + slot], 1)] = e;
}

// push_edge for N edges of each lane at once (-1: none): their exchanges are in flight together, and one atomic
// takes the positions of all of them.
template <int CAP, int N>
__device__ __forceinline__ void push_edges(const Topo &t, const int (&e)[N], int stamp, int slot, Stage<CAP> *st) {
    int old[N];
#pragma unroll
    for (int k = 0; k < N; ++k) old[k] = e[k] >= 0 ? atomicExch(&t.edge_stamp[e[k]], stamp) : stamp;
    unsigned long long m[N];
    int total = 0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        m[k] = __ballot(old[k] != stamp);
        total += __popcll(m[k]);
    }
    if (total == 0) return;   // the same in every active lane
    const int lane = __lane_id();
    const int leader = __ffsll((unsigned long long)__ballot(true)) - 1;
    int base = 0;
    if (lane == leader) base = atomicAdd(st ? &st->cnt : &t.ctl[K_WL + slot], total);
    base = __shfl(base, leader);
#pragma unroll
    for (int k = 0; k < N; ++k) {
        if (old[k] != stamp) {
            const int pos = base + __popcll(m[k] & ((1ull << lane) - 1ull));
            if (!st)
                wl_of(t, slot)[pos] = e[k];
            else if (pos < CAP)
                st->buf[pos] = e[k];
            else
                wl_of(t, slot)[atomicAdd(&t.ctl[K_WL + slot], 1)] = e[k];
        }
        base += __popcll(m[k]);
    }
}

// Is d already a neighbour of the finite vertex c?  A flip of (a, b) into
// (c, d) is only a flip if c-d is not an edge yet: on an embedded
// triangulation that always holds, but on a folded one (several inverted
// triangles around a disk that crossed more than one edge) the inverted-
// triangle rule can ask for it, and performing it would glue a duplicate edge.
// The star is read during evaluation, before any flip of the round.
// The two directions around c are walked at once: the walk is a chain of dependent loads, and this halves it.
__device__ __forceinline__ bool adjacent(const Topo &t, int c, int d) {
    const int h0 = t.vert_he[c];
    if (bad_he(t, h0)) return true;
    if (t.he_v[bd_next(h0)] == d) return true;
    int hf = h0, hb = h0, guard = 0;
    for (;;) {
        const int tf = t.he_twin[bd_prev(hf)], tb = t.he_twin[hb];
        if (bad_he(t, tf)) return true;
        if (tf == hb) return false;
        if (bad_he(t, tb)) return true;
        const int nb = bd_next(tb);
        if (t.he_v[bd_next(tf)] == d || t.he_v[bd_next(nb)] == d) return true;
        if (nb == tf) return false;
        if (++guard > 2048) return true;
        hf = tf;
        hb = nb;
    }
}

// Stars, one per kStarLanes lanes.  The star of a disk is its outgoing
// half-edges in counter-clockwise order from vert_he; lane q of the group holds
// half-edges q and q + kStarLanes with their far vertices.  Finding it is a
// chain of dependent loads (each half-edge from the one before), walked from
// both ends at once by the whole group (same addresses); everything after it is
// one load per lane.  Stars above kStarMax are left to one lane.  (Sixteen lanes
// in the one-workgroup tail, one half-edge each: 2% faster rounds below 64 stars,
// but twice the passes above: 272 against 247 us a step at 16,000 disks.)
constexpr int kStarLanes = 8;
constexpr int kStarMax = 2 * kStarLanes;
constexpr int kStarLarge = -1;

struct Star {
    int deg;         // kStarLarge: more than kStarMax; 0: the walk met an index out of range
    int h[2], w[2];
};
struct StarPos {   // positions of the disk and of the far vertices a lane holds
    double2 pv, pw[2];
};

__device__ __forceinline__ int star_base() { return (int)__lane_id() & ~(kStarLanes - 1); }
__device__ __forceinline__ int star_lane() { return (int)__lane_id() & (kStarLanes - 1); }
// Whether `any` holds in a lane of this lane's group (every lane of the group is here).
__device__ __forceinline__ bool star_any(bool any) {
    return ((__ballot(any) >> star_base()) & ((1ull << kStarLanes) - 1ull)) != 0;
}
// Value held for half-edge i of the star (two: some star of the wavefront has more than kStarLanes).
template <typename T>
__device__ __forceinline__ T star_get(const T (&x)[2], int i, bool two) {
    const int src = star_base() + (i & (kStarLanes - 1));
    const T a = __shfl(x[0], src);
    if (!two) return a;
    const T b = __shfl(x[1], src);
    return i < kStarLanes ? a : b;
}
__device__ __forceinline__ double2 star_get2(const double2 (&x)[2], int i, bool two) {
    double ax[2], ay[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        ax[u] = x[u].x;
        ay[u] = x[u].y;
    }
    return make_double2(star_get(ax, i, two), star_get(ay, i, two));
}
__device__ __forceinline__ bool star_two(const Star &s) { return __ballot(s.deg > kStarLanes) != 0; }

__device__ __forceinline__ Star star_walk(const Topo &t, int v) {
    Star s;
    s.deg = 0;
#pragma unroll
    for (int u = 0; u < 2; ++u) s.h[u] = s.w[u] = -1;
    const int q = star_lane();
    const int h0 = t.vert_he[v];
    if (bad_he(t, h0)) return s;
    int bh = -1, bw = -1;   // lane r: the r-th half-edge clockwise from vert_he
    int hf = h0, hb = h0, nf = 1, nb = 0;
    if (q == 0) {
        s.h[0] = h0;
        s.w[0] = t.he_v[bd_next(h0)];
    }
    for (;;) {
        const int tf = t.he_twin[bd_prev(hf)], tb = t.he_twin[hb];
        if (bad_he(t, tf)) return s;
        if (tf == hb) break;
        if (bad_he(t, tb)) return s;
        const int cw = bd_next(tb);
        const bool meet = cw == tf;
        if (nf + nb + (meet ? 1 : 2) > kStarMax) {
            s.deg = kStarLarge;
            return s;
        }
        if (q == (nf & (kStarLanes - 1))) {
            const int w = t.he_v[bd_next(tf)];
            if (nf < kStarLanes) {
                s.h[0] = tf;
                s.w[0] = w;
            } else {
                s.h[1] = tf;
                s.w[1] = w;
            }
        }
        ++nf;
        if (meet) break;
        if (q == nb) {
            bh = cw;
            bw = t.he_v[bd_next(cw)];
        }
        ++nb;
        hf = tf;
        hb = cw;
    }
    const int deg = nf + nb;
    bool ok = true;
#pragma unroll
    for (int u = 0; u < 2; ++u) {   // half-edge i >= nf is the (deg - 1 - i)-th clockwise one
        const int i = q + u * kStarLanes;
        const int src = star_base() + ((deg - 1 - i) & (kStarLanes - 1));
        const int h = __shfl(bh, src), w = __shfl(bw, src);
        if (i >= nf && i < deg) {
            s.h[u] = h;
            s.w[u] = w;
        }
        if (i < deg && bad_v(t, s.w[u])) ok = false;
    }
    s.deg = star_any(!ok) ? 0 : deg;
    return s;
}

// The star that the current round's gather recorded for the disk queued at idx; with `rewritten`, whether a flip
// round rfirst or later (absolute) rewrote the triangle of a half-edge this lane holds.  Two dependent loads deep:
// the record has room for kStarMax whatever the degree, and lanes past the degree read the tables' first entries.
__device__ __forceinline__ Star star_recorded(const Topo &t, int idx, int rfirst = 0, bool *rewritten = nullptr) {
    Star s;
    const int *rec = t.star + (size_t)idx * kStarMax + star_lane();
    s.deg = t.star_deg[idx];
    s.h[0] = rec[0];
    s.h[1] = -1;
    const bool two = star_two(s);
    if (two) s.h[1] = rec[kStarLanes];
    int w[2] = {-1, -1}, stamp[2] = {0, 0};
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        if (u == 1 && !two) continue;
        const int h = star_lane() + u * kStarLanes < s.deg ? s.h[u] : 0;
        w[u] = t.he_v[bd_next(h)];
        if (rewritten) stamp[u] = t.tri_stamp[h / 3];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const bool held = star_lane() + u * kStarLanes < s.deg;
        if (!held) s.h[u] = -1;
        s.w[u] = held ? w[u] : -1;
        if (rewritten && held && stamp[u] >= rfirst) *rewritten = true;
    }
    return s;
}

// Workgroup staging of flip candidates (LDS), for the full evaluation: lanes
// take stage positions with one LDS atomic per wavefront; at the end the
// workgroup reserves its candidates in the round's list with one atomic and
// copies them out (same-address atomics from every CU serialise).  Candidates
// beyond the stage's capacity go to the list directly.
template <int CAP>
struct CandStage {
    int2 buf[CAP];
    int cnt, base;
};

// The flip decision `rule` for the canonical edge h (twin tw, opposite vertices
// c and d): count an inverted quad; a flipping edge becomes a candidate of
// round slot `slot` and claims its two triangles.
template <int CAP = 1>
__device__ __forceinline__ void register_flip(const Topo &t, int h, int tw, int c, int d, int rule, bool inverted,
                                              int round, int slot, CandStage<CAP> *st = nullptr) {
    wave_count(&t.ctl[K_INVQ + slot], inverted);
    if (rule == BD_NOFLIP) return;
    if (c < t.inf ? adjacent(t, c, d) : adjacent(t, d, c)) {
        // blocked for now (c-d may disappear in this very round): look again next round
        push_edge(t, h, round + 1, slot + 1 == MAXR ? 0 : slot + 1);
        return;
    }
    const int t1 = h / 3, t2 = tw / 3;
    // an edge may be evaluated more than once in a round: the first evaluation is the one that does not find its
    // own claim.  An edge that finds a stronger claim cannot win this round and is looked at again in the next.
    const unsigned long long key = claim_key(round, h);
    const unsigned long long held = atomicMax(&t.claim[t1], key);
    if (held == key) return;
    atomicMax(&t.claim[t2], key);
    if (held > key) {
        push_edge(t, h, round + 1, slot + 1 == MAXR ? 0 : slot + 1);
        return;
    }
    const int2 cand = make_int2(h, t2 | (rule == BD_FLIP_INVERSION ? (int)0x80000000 : 0));
    if (st) {
        const int p = wave_reserve(&st->cnt, true);
        if (p < CAP)
            st->buf[p] = cand;
        else
            t.cand[atomicAdd(&t.ctl[K_CAND + slot], 1)] = cand;
    } else {
        t.cand[wave_reserve(&t.ctl[K_CAND + slot], true)] = cand;
    }
}

// Evaluates the canonical edge h (h < twin) and, if it must flip, registers
// it as a candidate of round slot `slot` and claims its two triangles.
template <int CAP, class TP>
__device__ __forceinline__ void eval_edge(const TP &t, int h, int tw, int round, int slot, CandStage<CAP> *st) {
    if (bad_he(t, tw)) return topo_err(t);
    const int a = t.he_v[h], b = t.he_v[bd_next(h)], c = t.he_v[bd_prev(h)];
    const int d = t.he_v[bd_prev(tw)];
    if (bad_v(t, a) || bad_v(t, b) || bad_v(t, c) || bad_v(t, d)) return topo_err(t);
    bool inverted = false;
    const int rule = flip_rule_at(t, a, b, c, d, t.xy[a], t.xy[b], t.xy[c], t.xy[d], &inverted);
    register_flip<CAP>(t, h, tw, c, d, rule, inverted, round, slot, st);
}

// Full evaluation after a move: one thread per triangle.  The triangle's three
// vertices and their positions are read once for its canonical edges (h <
// twin), and the far vertices of those edges are read together, so a thread
// issues its loads in three dependent waves instead of one chain per edge.
// The decisions are those of eval_edge.
constexpr int kEvalStage = 2048;
// Workgroup and grid of the full evaluation: bound by the rate of its scattered loads (some twenty a triangle), so by
// the wavefronts a compute unit holds.  80 registers let six wavefronts of a SIMD run, which workgroups of 1024
// threads cannot fill; five workgroups of 256 per compute unit are all resident at once.  1,000,000 disks 73 us as
// 512 x 1024, 66 so, 81 as 1536 x 256 (some wait for a place and run alone); 16,001 disks 16.0 and 11.5; 64 systems
// of 2,048 to 32,768 74 and 63.
constexpr int kEvalBlock = 256, kEvalGrid = 1280;

// Every thread of the workgroup calls it once, at the end: the staged
// candidates are reserved in the round's list with one atomic and copied out.
template <int CAP>
__device__ __forceinline__ void cand_flush(const Topo &t, int slot, CandStage<CAP> &st) {
    __syncthreads();
    const int n = st.cnt < CAP ? st.cnt : CAP;
    if (threadIdx.x == 0 && n > 0) st.base = atomicAdd(&t.ctl[K_CAND + slot], n);
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) t.cand[st.base + i] = st.buf[i];
}

// snap: where the topology is copied aside (v == null: not): the pass reads all of it anyway.
struct Snapshot {
    int *v, *twin, *vh;
    int nvh;
};

template <class TP>
__global__ __launch_bounds__(kEvalBlock) void k_flip_eval_full(TP t, int round, int slot, int reversal,
                                                               Snapshot snap) {
    __shared__ CandStage<kEvalStage> st;
    if (stopped(t.ctl)) return;   // nothing in this launch writes the stop flags: uniform
    if (snap.v)
        for (int i = xcd_block() * blockDim.x + threadIdx.x; i < snap.nvh; i += gridDim.x * blockDim.x)
            snap.vh[i] = t.vert_he[i];
    if (threadIdx.x == 0) st.cnt = 0;
    __syncthreads();
    round += t.base->rbase;
    for (int tri = xcd_block() * blockDim.x + threadIdx.x; tri < t.T; tri += gridDim.x * blockDim.x) {
        const int h0 = 3 * tri;
        int v[3], tw[3], d[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            v[k] = t.he_v[h0 + k];
            tw[k] = t.he_twin[h0 + k];
        }
        if (snap.v) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                snap.v[h0 + k] = v[k];
                snap.twin[h0 + k] = tw[k];
            }
        }
        bool own[3], ok = true;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            own[k] = h0 + k < tw[k];
            if (own[k] && bad_he(t, tw[k])) own[k] = false, ok = false;
            d[k] = own[k] ? t.he_v[bd_prev(tw[k])] : v[k];
            if (bad_v(t, v[k]) || bad_v(t, d[k])) ok = false;
        }
        if (!ok) {
            topo_err(t);
            continue;
        }
        double px[3], py[3], qx[3], qy[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double2 pv = t.xy[v[k]];
            px[k] = pv.x;
            py[k] = pv.y;
            if (own[k]) {   // the far vertex of a canonical edge (the others are not evaluated here)
                const double2 pd = t.xy[d[k]];
                qx[k] = pd.x;
                qy[k] = pd.y;
            } else {
                qx[k] = pv.x;
                qy[k] = pv.y;
            }
        }
        if (reversal) {
            double ox[3], oy[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                ox[k] = t.xo[v[k]];
                oy[k] = t.yo[v[k]];
            }
            // Sec. 4.3: the pair passed through each other if the edge vector reversed
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int k1 = k == 2 ? 0 : k + 1;
                bool rev = false;
                if (own[k] && v[k] < t.n && v[k1] < t.n) {
                    const double rx = sep_p(t, ox[k1] - ox[k]), ry = sep_p(t, oy[k1] - oy[k]);
                    const double mx = sep_p(t, px[k1] - px[k]), my = sep_p(t, py[k1] - py[k]);
                    rev = rx * mx + ry * my < 0.0;
                }
                wave_count64(&t.acc[A_REVERSALS], rev);
                if (reversal == 2) wave_count(&t.ctl[K_REV], rev);
            }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (!own[k]) continue;
            const int k1 = k == 2 ? 0 : k + 1, k2 = k == 0 ? 2 : k - 1;
            const int a = v[k], b = v[k1], c = v[k2];
            bool inverted = false;
            int rule;
            if (TP::kPer) {
                const double ax = px[k], ay = py[k];
                rule = bd_flip_rule_quad(0.0, 0.0, sep_p(t, px[k1] - ax), sep_p(t, py[k1] - ay),
                                         sep_p(t, px[k2] - ax), sep_p(t, py[k2] - ay), sep_p(t, qx[k] - ax),
                                         sep_p(t, qy[k] - ay), true, &inverted);
            } else {
                rule = bd_flip_rule_xy(a, b, c, d[k], t.inf, px[k], py[k], px[k1], py[k1], px[k2], py[k2], qx[k],
                                       qy[k], true, &inverted);
            }
            register_flip<kEvalStage>(t, h0 + k, tw[k], c, d[k], rule, inverted, round, slot, &st);
        }
    }
    cand_flush(t, slot, st);
}

template <int CAP, class TP>
__device__ __forceinline__ void flip_eval_list_body(const TP &t, int round, int slot, int i0, int stride,
                                                    CandStage<CAP> *st) {
    if (stopped(t.ctl)) return;
    round += t.base->rbase;
    const int count = t.ctl[K_WL + slot];
    const int *wl = wl_of(t, slot);
    for (int idx = i0; idx < count; idx += stride) {
        int h = wl[idx];
        if (bad_he(t, h)) {
            topo_err(t);
            continue;
        }
        int tw = t.he_twin[h];
        if (bad_he(t, tw)) {
            topo_err(t);
            continue;
        }
        if (tw < h) {
            int s = h;
            h = tw;
            tw = s;
        }
        eval_edge<CAP>(t, h, tw, round, slot, st);
    }
}

template <class TP>
__global__ void k_flip_eval_list(TP t, int round, int slot) {
    __shared__ CandStage<kEvalStage> st;
    if (stopped(t.ctl)) return;   // nothing in this launch writes the stop flags: uniform
    if (threadIdx.x == 0) st.cnt = 0;
    __syncthreads();
    flip_eval_list_body<kEvalStage>(t, round, slot, xcd_block() * blockDim.x + threadIdx.x, gridDim.x * blockDim.x,
                                    &st);
    cand_flush(t, slot, st);
}

// Evaluates the edges of the triangles at disk v (star s) and loads its positions.  False when an index was out of
// range, or for a star above kStarMax (evaluated here by one lane): then the positions are not loaded.  The edge to
// a far vertex and the one across from the disk go through one copy of the flip rule, in canonical order.
template <int CAP, class TP>
__device__ __forceinline__ bool eval_star(const TP &t, int v, const Star &s, int round, int slot,
                                          StarPos &sp, CandStage<CAP> *st) {
    const int q = star_lane();
    if (s.deg == kStarLarge) {
        if (q != 0) return false;
        const int h0 = t.vert_he[v];
        if (bad_he(t, h0)) {
            topo_err(t);
            return false;
        }
        int h = h0, guard = 0;
        do {
#pragma clang loop unroll(disable)
            for (int e = 0; e < 2; ++e) {
                const int l = e ? bd_next(h) : h, lt = t.he_twin[l];
                if (bad_he(t, lt))
                    topo_err(t);
                else
                    eval_edge<CAP>(t, l < lt ? l : lt, l < lt ? lt : l, round, slot, st);
            }
            h = t.he_twin[bd_prev(h)];
            if (bad_he(t, h)) {
                topo_err(t);
                break;
            }
        } while (h != h0 && ++guard < 4096);
        return false;
    }
    const int deg = s.deg;
    const bool two = star_two(s);
    const double2 pv = t.xy[v];
    sp.pv = pv;
    int lt[2], far[2];
    double2 pf[2];
    bool ok = true;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        lt[u] = far[u] = -1;
        sp.pw[u] = pf[u] = pv;
        if (q + u * kStarLanes >= deg) continue;
        lt[u] = t.he_twin[bd_next(s.h[u])];
        if (bad_v(t, s.w[u]))
            ok = false;
        else
            sp.pw[u] = t.xy[s.w[u]];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        if (q + u * kStarLanes >= deg) continue;
        if (bad_he(t, lt[u]))
            ok = false;
        else
            far[u] = t.he_v[bd_prev(lt[u])];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        if (q + u * kStarLanes >= deg || !ok) continue;
        if (bad_v(t, far[u]))
            ok = false;
        else
            pf[u] = t.xy[far[u]];
    }
    if (!ok) topo_err(t);
    if (star_any(!ok)) return false;   // the group's lanes are here together
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        if (u == 1 && !two) continue;
        const int i = q + u * kStarLanes;
        const int ip = i + 1 >= deg ? 0 : i + 1, im = i == 0 ? deg - 1 : i - 1;
        const int wn = star_get(s.w, ip, two), wp = star_get(s.w, im, two), hp = star_get(s.h, im, two);
        const double2 pn = star_get2(sp.pw, ip, two), pp = star_get2(sp.pw, im, two);
        if (i >= deg) continue;
#pragma clang loop unroll(disable)
        for (int e = 0; e < 2; ++e) {
            // e = 0: v - w_i, triangles (v, w_i, w_(i+1)) and (w_i, v, w_(i-1)); e = 1: w_i - w_(i+1), triangles
            // (w_i, w_(i+1), v) and (w_(i+1), w_i, far)
            const int h = e ? bd_next(s.h[u]) : s.h[u], g = e ? lt[u] : bd_prev(hp);
            const bool fwd = h < g;
            const int a0 = e ? s.w[u] : v, b0 = e ? wn : s.w[u], c0 = e ? v : wn, d0 = e ? far[u] : wp;
            const double2 pa0 = e ? sp.pw[u] : pv, pb0 = e ? pn : sp.pw[u], pc0 = e ? pv : pn, pd0 = e ? pf[u] : pp;
            const int c = fwd ? c0 : d0, d = fwd ? d0 : c0;
            bool inverted = false;
            const int rule = flip_rule_at(t, fwd ? a0 : b0, fwd ? b0 : a0, c, d, fwd ? pa0 : pb0, fwd ? pb0 : pa0,
                                          fwd ? pc0 : pd0, fwd ? pd0 : pc0, &inverted);
            register_flip<CAP>(t, fwd ? h : g, fwd ? g : h, c, d, rule, inverted, round, slot, st);
        }
    }
    return true;
}

// First evaluation of the repair after overlap round k: every edge of the triangles at the disks the round moved,
// from the stars its gather recorded (the topology has not changed since).  Lane i of a star takes the edge to
// its far vertex w_i and the edge w_i - w_(i+1) across from the disk.  No worklist: an edge of two moved disks is
// evaluated by both.  65,536 disks: 17 us for the walk that queued the edges and 8 us for their evaluation before.
template <class TP>
__global__ __launch_bounds__(256) void k_flip_eval_star(TP t, int k, int round, int slot) {
    __shared__ CandStage<kEvalStage> st;
    if (stopped(t.ctl)) return;   // nothing in this launch writes the stop flags: uniform
    if (threadIdx.x == 0) st.cnt = 0;
    __syncthreads();
    const int i0 = xcd_block() * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    const int ntouched = t.ctl[K_TOUCH + k];
    const int *touched = touched_of(t, k);
    flip_eval_list_body<kEvalStage>(t, round, slot, i0, stride, &st);   // edges the repair before left blocked
    for (int g = i0 / kStarLanes; g < ntouched; g += stride / kStarLanes) {
        StarPos sp;
        eval_star<kEvalStage>(t, touched[g], star_recorded(t, g), round + t.base->rbase, slot, sp, &st);
    }
    cand_flush(t, slot, st);
}

__device__ __forceinline__ void flip_apply_body(const Topo &t, int round, int slot, int i0, int stride) {
    round += t.base->rbase;
    if (stopped(t.ctl)) return;
    const int ncand = t.ctl[K_CAND + slot];
    const int epoch = t.ctl[K_FL_EPOCH];
    for (int idx = i0; idx < ncand; idx += stride) {
        const int2 cd = t.cand[idx];
        const int h = cd.x, t1 = h / 3, t2 = cd.y & 0x7FFFFFFF;
        const unsigned long long key = claim_key(round, h);
        const bool won = t.claim[t1] == key && t.claim[t2] == key;
        t.cand_won[idx] = 0;
        if (!won) continue;
        // the quad is owned by this thread: (a, b, c) = t1 from h, (b, a, d) = t2 from its twin
        const int hb = bd_next(h), hc = bd_prev(h);
        const int g = t.he_twin[h];
        if (g / 3 != t2) {
            topo_err(t);
            continue;
        }
        const int ga = bd_next(g), gd = bd_prev(g);
        const int a = t.he_v[h], b = t.he_v[hb], c = t.he_v[hc], d = t.he_v[gd];
        const int Thb = t.he_twin[hb], Thc = t.he_twin[hc], Tga = t.he_twin[ga], Tgd = t.he_twin[gd];
        if (bad_v(t, a) || bad_v(t, b) || bad_v(t, c) || bad_v(t, d) || bad_he(t, Thb) || bad_he(t, Thc) ||
            bad_he(t, Tga) || bad_he(t, Tgd)) {
            topo_err(t);
            continue;
        }
        const int s1 = 3 * t1, s2 = 3 * t2;
        // new t1 = (c, a, d), new t2 = (d, b, c); the diagonal c-d is slot 2 of both
        t.he_v[s1 + 0] = c;
        t.he_v[s1 + 1] = a;
        t.he_v[s1 + 2] = d;
        t.he_v[s2 + 0] = d;
        t.he_v[s2 + 1] = b;
        t.he_v[s2 + 2] = c;
        t.he_twin[s1 + 0] = Thc;   // c -> a, old neighbour index (fixed in k_flip_fix)
        t.he_twin[s1 + 1] = Tga;   // a -> d
        t.he_twin[s1 + 2] = s2 + 2;
        t.he_twin[s2 + 0] = Tgd;   // d -> b
        t.he_twin[s2 + 1] = Thb;   // b -> c
        t.he_twin[s2 + 2] = s1 + 2;
        t.moved[hc] = s1 + 0;
        t.moved[ga] = s1 + 1;
        t.moved[gd] = s2 + 0;
        t.moved[hb] = s2 + 1;
        t.tri_stamp[t1] = round;
        t.tri_stamp[t2] = round;
        // every flip rewrites the outgoing half-edge of all four vertices, so each
        // entry stays valid whichever concurrent flip writes it last
        t.vert_he[a] = s1 + 1;
        t.vert_he[b] = s2 + 1;
        t.vert_he[c] = s1 + 0;
        t.vert_he[d] = s2 + 0;
        t.cand_won[idx] = 1;
        // the new diagonal joins two disks that may never have been tested for overlap
        const int e = s1 + 2 < s2 + 2 ? s1 + 2 : s2 + 2;
        // and both rewritten triangles go to the validation that ends the repair (the exchanges, then the two
        // counters, are in flight together: each is a round trip to the L2)
        const int old_e = atomicExch(&t.fl_stamp[e], epoch);
        const int old_1 = atomicExch(&t.vt_stamp[t1], epoch), old_2 = atomicExch(&t.vt_stamp[t2], epoch);
        const unsigned long long me = __ballot(old_e != epoch), m1 = __ballot(old_1 != epoch),
                                 m2 = __ballot(old_2 != epoch), lt = (1ull << __lane_id()) - 1ull;
        const int leader = __ffsll((unsigned long long)__ballot(true)) - 1;
        int be = 0, bt = 0;
        if (__lane_id() == leader) {
            be = atomicAdd(&t.ctl[K_FL_N], __popcll(me));
            bt = atomicAdd(&t.ctl[K_VT_N], __popcll(m1) + __popcll(m2));
        }
        be = __shfl(be, leader);
        bt = __shfl(bt, leader);
        if (old_e != epoch) t.fl[be + __popcll(me & lt)] = e;
        if (old_1 != epoch) t.vt[bt + __popcll(m1 & lt)] = t1;
        if (old_2 != epoch) t.vt[bt + __popcll(m1) + __popcll(m2 & lt)] = t2;
        wave_count64(&t.acc[A_FLIPS], true);
        wave_count64(&t.acc[A_INV_FLIPS], (cd.y & (int)0x80000000) != 0);
    }
}

__global__ void k_flip_apply(Topo t, int round, int slot) {
    flip_apply_body(t, round, slot, xcd_block() * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

template <int CAP = 1>
__device__ __forceinline__ void flip_fix_body(const Topo &t, int round, int slot, int i0, int stride,
                                              Stage<CAP> *st = nullptr) {
    round += t.base->rbase;
    if (stopped(t.ctl)) return;
    const int ncand = t.ctl[K_CAND + slot];
    const int next = round + 1;
    const int nslot = slot + 1 == MAXR ? 0 : slot + 1;   // slots are used circularly
    for (int idx = i0; idx < ncand; idx += stride) {
        const int2 cd = t.cand[idx];
        const int h = cd.x, t1 = h / 3, t2 = cd.y & 0x7FFFFFFF;
        // the edges to queue: a flip's four outer edges and its diagonal, or the candidate itself when it lost
        // and neither of its triangles flipped (loads, exchanges and list positions of the five taken together)
        int e[5] = {-1, -1, -1, -1, -1};
        if (!t.cand_won[idx]) {
            if (t.tri_stamp[t1] != round && t.tri_stamp[t2] != round) e[4] = h;
        } else {
            const int outer[4] = {3 * t1 + 0, 3 * t1 + 1, 3 * t2 + 0, 3 * t2 + 1};
            int o[4], mv[4], ts[4];
            bool ok[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                o[k] = t.he_twin[outer[k]];
                ok[k] = !bad_he(t, o[k]);
                if (!ok[k]) topo_err(t);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                ts[k] = ok[k] ? t.tri_stamp[o[k] / 3] : 0;
                mv[k] = ok[k] ? t.moved[o[k]] : 0;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (!ok[k]) continue;
                int tw = o[k];
                if (ts[k] == round) {
                    tw = mv[k];
                    if (bad_he(t, tw)) {
                        topo_err(t);
                        continue;
                    }
                    t.he_twin[outer[k]] = tw;
                } else {
                    t.he_twin[tw] = outer[k];
                }
                e[k] = outer[k] < tw ? outer[k] : tw;
            }
            const int d1 = 3 * t1 + 2, d2 = 3 * t2 + 2;
            e[4] = d1 < d2 ? d1 : d2;
        }
        push_edges<CAP, 5>(t, e, next, nslot, st);
    }
}

constexpr int kFixStage = 2048;

__global__ void k_flip_fix(Topo t, int round, int slot) {
    __shared__ Stage<kFixStage> st;
    if (stopped(t.ctl)) return;   // nothing in this launch writes the stop flags: uniform
    stage_init(st);
    flip_fix_body(t, round, slot, xcd_block() * blockDim.x + threadIdx.x, gridDim.x * blockDim.x, &st);
    const int nslot = slot + 1 == MAXR ? 0 : slot + 1;
    stage_flush(st, &t.ctl[K_WL + nslot], wl_of(t, nslot));
}

// Counts finite triangles that are not positively oriented after repair `rep`.
// inv: the repair's invalid-triangle counter, or a workgroup's share of it in LDS
template <class TP>
__device__ __forceinline__ void validate_tri(const TP &t, int tri, int *inv) {
    const int a = t.he_v[3 * tri], b = t.he_v[3 * tri + 1], c = t.he_v[3 * tri + 2];
    if (bad_v(t, a) || bad_v(t, b) || bad_v(t, c)) {
        atomicAdd(inv, 1);
        topo_err(t);
        return;
    }
    if (a >= t.inf || b >= t.inf || c >= t.inf) return;
    if (orient_at(t, t.xy[a], t.xy[b], t.xy[c]) <= 0.0) atomicAdd(inv, 1);
}

// End of repair `rep` whose last round used slot `last`: halt the step when the
// repair did not finish inside its round budget or left an invalid triangle.
__device__ __forceinline__ void repair_check_body(int *ctl, int rep, int last) {
    if (stopped(ctl)) return;
    int reason = 0;
    if (ctl_read(ctl, K_TOPO) != 0)
        reason = HALT_TOPOLOGY;
    else if (ctl_read(ctl, K_REV) != 0)   // only ever set by a move whose reversals halve the step
        reason = HALT_REVERSAL;
    else if (ctl_read(ctl, K_CAND + last) != 0)
        reason = HALT_REPAIR_BUDGET;
    else if (ctl_read(ctl, K_INV + rep) != 0)
        reason = HALT_INVALID;
    if (reason) {
        ctl[K_REASON] = reason;
        ctl[K_STAGE] = rep;
        ctl[K_LAST] = last;
        ctl[K_HALT] = 1;
    }
}

// Adds a workgroup's count (in LDS) to a shared counter from thread 0; every
// thread calls it.  Returns true in thread 0 when it added something.
__device__ __forceinline__ bool add_block_count(int *counter, const int *block_count) {
    __syncthreads();
    if (threadIdx.x != 0 || *block_count == 0) return false;
    atomicAdd(counter, *block_count);
    return true;
}

template <class TP>
__global__ __launch_bounds__(kScanBlock) void k_validate(TP t, int rep) {
    __shared__ int inv;
    if (stopped(t.ctl)) return;   // nothing in this launch writes the stop flags: uniform
    if (threadIdx.x == 0) inv = 0;
    __syncthreads();
    for (int tri = xcd_block() * blockDim.x + threadIdx.x; tri < t.T; tri += gridDim.x * blockDim.x)
        validate_tri(t, tri, &inv);
    add_block_count(&t.ctl[K_INV + rep], &inv);
}

// ---------------------------------------------------------------- overlaps
// Detect: every Delaunay edge between two disks with d < (r_i + r_j)(1 - tol)
// (Algorithm 2 test, Sec. 2.3 contact distance); both ends are queued once
// per round.
__device__ __forceinline__ void ovl_check_body(int *ctl, int k, int stamp, const StepBase *base);
__device__ __forceinline__ void final_check_body(int *ctl, int k);

// Full detection.  A step's first detection finds tens of thousands of
// overlapping pairs on a large system; the disks it marks are staged in the
// workgroup's LDS and copied out with one reservation on the shared counter
// per kDetStage entries, not one per wavefront and edge (same-address
// atomics from every CU serialise and dominated this scan).
constexpr int kDetBlock = kScanBlock;
constexpr int kDetStage = 16384;   // 64 KiB of LDS
constexpr int kDetPerIter = 6 * kDetBlock;   // at most two disks for each of three edges per thread

__device__ __forceinline__ void det_flush(const Topo &t, int k, int *buf, int &cnt, int &base) {
    // every thread of the workgroup is here, after a barrier
    if (threadIdx.x == 0) base = atomicAdd(&t.ctl[K_TOUCH + k], cnt);
    __syncthreads();
    int *out = touched_of(t, k) + base;
    for (int i = threadIdx.x; i < cnt; i += kDetBlock) out[i] = buf[i];
    __syncthreads();
    if (threadIdx.x == 0) cnt = 0;
    __syncthreads();
}

// vrep >= 0: the same pass also validates every triangle for the repair in
// slot vrep (last round slot vlast), whose check the last workgroup runs
// before the detection's.
template <class TP>
__global__ __launch_bounds__(kDetBlock) void k_ovl_detect(TP t, int rstamp, double keep, int k, int check, int vrep,
                                                          int vlast) {
#pragma clang fp contract(off)
    __shared__ int buf[kDetStage];
    __shared__ int cnt, base, nfound, inv;
    if (stopped(t.ctl)) return;   // nothing in this launch writes the stop flags before its last workgroup
    const int stamp = rstamp + t.base->vbase;
    if (threadIdx.x == 0) {
        cnt = 0;
        nfound = 0;
        inv = 0;
    }
    __syncthreads();
    int found = 0;
    for (int t0 = xcd_block() * kDetBlock; t0 < t.T; t0 += gridDim.x * kDetBlock) {   // same trip count for the workgroup
        const int tri = t0 + threadIdx.x;
        if (tri < t.T) {
            // the triangle's vertices, positions and radii read once for its validation and its
            // canonical edges
            int v[3], tw[3];
            double px[3], py[3], pr[3];
            bool ok = true;
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                v[e] = t.he_v[3 * tri + e];
                tw[e] = t.he_twin[3 * tri + e];
                if (bad_v(t, v[e])) ok = false;
            }
            if (!ok) topo_err(t);
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                const bool fin = ok && v[e] < t.inf;
                const double2 pv = fin ? t.xy[v[e]] : make_double2(0.0, 0.0);
                px[e] = pv.x;
                py[e] = pv.y;
                pr[e] = fin ? (t.ru > 0.0 ? t.ru : t.rad[v[e]]) : 0.0;
            }
            if (vrep >= 0) {   // as validate_tri
                if (!ok) {
                    atomicAdd(&inv, 1);
                } else if (v[0] < t.inf && v[1] < t.inf && v[2] < t.inf) {
                    const double o = orient_at(t, make_double2(px[0], py[0]), make_double2(px[1], py[1]),
                                               make_double2(px[2], py[2]));
                    if (o <= 0.0) atomicAdd(&inv, 1);
                }
            }
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                const int h = 3 * tri + e;
                const int e1 = e == 2 ? 0 : e + 1;
                if (!ok || h > tw[e]) continue;
                const int a = v[e], b = v[e1];
                if (a >= t.n || b >= t.n) continue;
                const double dx = sep_p(t, px[e] - px[e1]), dy = sep_p(t, py[e] - py[e1]);
                const double d = sqrt(dx * dx + dy * dy);
                if (d < (pr[e] + pr[e1]) * keep) {
                    ++found;
                    const bool fa = atomicExch(&t.vstamp[a], stamp) != stamp;
                    const bool fb = atomicExch(&t.vstamp[b], stamp) != stamp;
                    if (fa || fb) {
                        int p = atomicAdd(&cnt, (fa ? 1 : 0) + (fb ? 1 : 0));
                        if (fa) buf[p++] = a;
                        if (fb) buf[p] = b;
                    }
                }
            }
        }
        __syncthreads();
        if (cnt > kDetStage - kDetPerIter) det_flush(t, k, buf, cnt, base);
    }
    for (int off = 32; off > 0; off >>= 1) found += __shfl_xor(found, off);
    if (__lane_id() == 0 && found) atomicAdd(&nfound, found);
    __syncthreads();
    if (cnt > 0) det_flush(t, k, buf, cnt, base);
    const bool a_ovl = threadIdx.x == 0 && nfound != 0;
    if (a_ovl) atomicAdd(&t.ctl[K_OVL + k], nfound);
    const bool a_inv = vrep >= 0 && add_block_count(&t.ctl[K_INV + vrep], &inv);
    if (check == 0) return;
    if (last_workgroup(t.ctl, a_ovl || a_inv) && threadIdx.x == 0) {
        if (vrep >= 0) repair_check_body(t.ctl, vrep, vlast);
        ovl_check_body(t.ctl, k, rstamp, t.base);
        if (check == 2) final_check_body(t.ctl, k);
    }
}

// Detection after overlap round kprev of the same step.  A Delaunay edge can
// only overlap now if one of its disks moved in round kprev (every disk of an
// edge that overlapped at round kprev's detection moved) or if a flip since
// that detection created it; every other edge was tested then and neither of
// its disks has moved.  So only the stars of the disks moved by round kprev
// and the flipped list are tested; an overlapping edge counts once (det_stamp).
// An overlapping edge (canonical id e): counted the first time it is found, both disks queued for overlap round k
// once per stamp.  With a workgroup stage (large rounds) the disks are marked only by the first to find the edge:
// 30 us for a round of 1,000,000 disks with all three exchanges issued together, 22 us so.  Without one (the tail)
// the exchanges are in flight together, since a round there waits for its chains.
template <int CAP>
__device__ __forceinline__ void found_edge(const Topo &t, int e, int a, int b, int stamp, int k, int &found,
                                           Stage<CAP> *st) {
    const int old_e = atomicExch(&t.det_stamp[e], stamp);
    int old_a = stamp, old_b = stamp;
    if (!st || old_e != stamp) {
        old_a = atomicExch(&t.vstamp[a], stamp);
        old_b = atomicExch(&t.vstamp[b], stamp);
    }
    if (old_e != stamp) ++found;
    const unsigned long long ma = __ballot(old_a != stamp), mb = __ballot(old_b != stamp);
    if ((ma | mb) == 0) return;
    const int lane = __lane_id(), leader = __ffsll((unsigned long long)__ballot(true)) - 1;
    const unsigned long long lt = (1ull << lane) - 1ull;
    int *counter = &t.ctl[K_TOUCH + k], *list = touched_of(t, k);
    int base = 0;
    if (lane == leader) base = atomicAdd(st ? &st->cnt : counter, __popcll(ma) + __popcll(mb));
    base = __shfl(base, leader);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        if (u == 0 ? old_a == stamp : old_b == stamp) continue;
        const int v = u == 0 ? a : b;
        const int pos = base + (u == 0 ? __popcll(ma & lt) : __popcll(ma) + __popcll(mb & lt));
        if (!st)
            list[pos] = v;
        else if (pos < CAP)
            st->buf[pos] = v;
        else
            list[atomicAdd(counter, 1)] = v;
    }
}

template <int CAP, class TP>
__device__ __forceinline__ void detect_edge(const TP &t, int h, int stamp, double keep, int k, int &found,
                                            Stage<CAP> *st) {
    const int tw = t.he_twin[h];
    if (bad_he(t, tw)) return topo_err(t);
    const int e = h < tw ? h : tw;
    const int a = t.he_v[e], b = t.he_v[bd_next(e)];
    if (bad_v(t, a) || bad_v(t, b)) return topo_err(t);
    if (a >= t.n || b >= t.n) return;
    const double2 pa = t.xy[a], pb = t.xy[b];
    const double dx = sep_p(t, pa.x - pb.x), dy = sep_p(t, pa.y - pb.y);
    const double d = sqrt(dx * dx + dy * dy);
    if (d < (t.ru > 0.0 ? t.ru + t.ru : t.rad[a] + t.rad[b]) * keep) found_edge(t, e, a, b, stamp, k, found, st);
}

// The validation of the repair after overlap round k fused with the next
// detection (round knew): both walk the stars of the disks round k moved, so
// one walk checks each triangle's orientation and tests each edge; then the
// triangles flips rewrote (validation) and the diagonals they created
// (detection).  The last workgroup runs the repair's check, then the
// detection's (check = 1) and the final check (check = 2).  On a repair that
// fails its check the detection's marks are never read: the host continues
// with rounds of its own slots and stamps.
// inv is the repair's invalid-triangle counter, or a workgroup's share of it in LDS; stamps are absolute here.

// The tests of one star: does the triangle after half-edge i, tested from its first half-edge on, not turn
// counter-clockwise; does the disk overlap the far one.
enum { STAR_INVALID = 1, STAR_HIT = 4 };   // shifted by u for half-edge q + u * kStarLanes

template <class TP>
__device__ __forceinline__ int star_test(const TP &t, int v, const Star &s, const StarPos &sp, double keep) {
#pragma clang fp contract(off)
    const int q = star_lane();
    const bool two = star_two(s);
    const double rv = t.ru > 0.0 ? t.ru : t.rad[v];
    const double2 pv = sp.pv;
    int r = 0;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        if (u == 1 && !two) continue;
        const int i = q + u * kStarLanes;
        const int ip = i + 1 >= s.deg ? 0 : i + 1;
        const int wn = star_get(s.w, ip, two);
        const double2 pn = star_get2(sp.pw, ip, two);
        if (i >= s.deg) continue;
        const int w = s.w[u];
        const double2 pw = sp.pw[u];
        if (w < t.inf && wn < t.inf) {   // the triangle (v, w, wn)
            const int f = s.h[u] % 3;
            const double o = orient_at(t, f == 0 ? pv : f == 1 ? pn : pw, f == 0 ? pw : f == 1 ? pv : pn,
                                       f == 0 ? pn : f == 1 ? pw : pv);
            if (o <= 0.0) r |= STAR_INVALID << u;
        }
        if (w < t.n) {
            const double dx = sep_p(t, pv.x - pw.x), dy = sep_p(t, pv.y - pw.y);
            const double d = sqrt(dx * dx + dy * dy);
            if (d < (rv + (t.ru > 0.0 ? t.ru : t.rad[w])) * keep) r |= STAR_HIT << u;
        }
    }
    return r;
}

// Commits the tests of a star: the repair's invalid count, the overlapping edges and their disks.
template <int CAP>
__device__ __forceinline__ void star_commit(const Topo &t, int v, const Star &s, int r, int *inv, int st,
                                            int knew, int &found, Stage<CAP> *stage) {
    const bool two = star_two(s);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        if (u == 1 && !two) continue;
        const int i = star_lane() + u * kStarLanes;
        const int tw = bd_prev(star_get(s.h, i == 0 ? s.deg - 1 : i - 1, two));   // the edge's other half
        if (r & (STAR_INVALID << u)) atomicAdd(inv, 1);
        if (r & (STAR_HIT << u))
            found_edge(t, s.h[u] < tw ? s.h[u] : tw, v, s.w[u], st, knew, found, stage);
    }
}

// A star above kStarMax, by one lane.
template <int CAP, class TP>
__device__ __forceinline__ void star_large(const TP &t, int v, int *inv, int st, double keep, int knew, int &found,
                                           Stage<CAP> *stage) {
    const int h0 = t.vert_he[v];
    int h = h0, guard = 0;
    do {
        validate_tri(t, h / 3, inv);
        detect_edge(t, h, st, keep, knew, found, stage);
        h = t.he_twin[bd_prev(h)];
        if (bad_he(t, h) || ++guard > 4096) {
            atomicAdd(inv, 1);
            topo_err(t);
            break;
        }
    } while (h != h0);
}

// Star of the disk queued at idx after the repair: as recorded where no flip of the repair (rounds rfirst and
// later, absolute) rewrote one of its triangles, else walked again; then its positions and its tests (r).  False
// when it was handled here (above kStarMax, by one lane; an index out of range).
template <int CAP, class TP>
__device__ __forceinline__ bool star_after_repair(const TP &t, int idx, int v, int *inv, int rfirst, int st,
                                                  double keep, int knew, int &found, Stage<CAP> *stage, Star &s,
                                                  int &r) {
    const int q = star_lane();
    bool rewritten = false;
    s = star_recorded(t, idx, rfirst, &rewritten);
    if (star_any(rewritten || s.deg <= 0)) s = star_walk(t, v);
    if (s.deg == kStarLarge) {
        if (q == 0) star_large(t, v, inv, st, keep, knew, found, stage);
        return false;
    }
    StarPos sp;
    sp.pv = t.xy[v];
    bool bad = s.deg == 0;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        sp.pw[u] = sp.pv;
        if (q + u * kStarLanes >= s.deg) continue;
        if (bad_v(t, s.w[u]))
            bad = true;
        else
            sp.pw[u] = t.xy[s.w[u]];
    }
    if (star_any(bad)) {
        if (q == 0) {
            atomicAdd(inv, 1);
            topo_err(t);
        }
        return false;
    }
    r = star_test(t, v, s, sp, keep);
    return true;
}

// The triangles and diagonals flips rewrote since the last detection.
template <int CAP, class TP>
__device__ __forceinline__ int validate_detect_flipped(const TP &t, int *inv, int st, double keep, int knew, int i0,
                                                       int stride, Stage<CAP> *stage) {
    const int nvt = t.ctl[K_VT_N], nfl = t.ctl[K_FL_N];
    int found = 0;
    for (int idx = i0; idx < nvt + nfl; idx += stride) {
        if (idx >= nvt) {
            const int e = t.fl[idx - nvt];
            if (bad_he(t, e))
                topo_err(t);
            else
                detect_edge(t, e, st, keep, knew, found, stage);
            continue;
        }
        const int tri = t.vt[idx];
        if ((unsigned)tri >= (unsigned)t.T)
            topo_err(t);
        else
            validate_tri(t, tri, inv);
    }
    return found;
}

constexpr int kTouchStage = 2048;

// One lane per edge and triangle of a star: 65,536 disks 11 us, 23 us as one thread per star, which exchanged a
// stamp per edge.
template <class TP>
__global__ __launch_bounds__(256) void k_validate_detect_local(TP t, int rep, int k, int rfirst, int last, int stamp,
                                                               double keep, int knew, int check) {
    __shared__ int inv, nfound;
    __shared__ Stage<kTouchStage> st;
    if (stopped(t.ctl)) return;   // nothing in this launch writes the stop flags before its last workgroup
    if (threadIdx.x == 0) {
        inv = 0;
        nfound = 0;
    }
    stage_init(st);
    const int i0 = xcd_block() * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    const int nmoved = t.ctl[K_TOUCH + k], vst = stamp + t.base->vbase;
    const int *moved = touched_of(t, k);
    int found = 0;
    // before the stars: their counts lie beside the counters that the workgroups add to as they end, and read late
    // they wait behind those atomics (1,000,000 disks, first round: 42 us with this pass last, 28 us so)
    found += validate_detect_flipped(t, &inv, vst, keep, knew, i0, stride, &st);
    for (int g = i0 / kStarLanes; g < nmoved; g += stride / kStarLanes) {
        const int v = moved[g];
        Star s;
        int r;
        if (star_after_repair(t, g, v, &inv, rfirst + t.base->rbase, vst, keep, knew, found, &st, s, r))
            star_commit(t, v, s, r, &inv, vst, knew, found, &st);
    }
    stage_flush(st, &t.ctl[K_TOUCH + knew], touched_of(t, knew));
    for (int off = 32; off > 0; off >>= 1) found += __shfl_xor(found, off);
    if (__lane_id() == 0 && found) atomicAdd(&nfound, found);
    const bool a1 = add_block_count(&t.ctl[K_INV + rep], &inv);
    const bool a2 = add_block_count(&t.ctl[K_OVL + knew], &nfound);
    if (last_workgroup(t.ctl, a1 || a2) && threadIdx.x == 0) {
        repair_check_body(t.ctl, rep, last);
        ovl_check_body(t.ctl, knew, stamp, t.base);
        if (check == 2) final_check_body(t.ctl, knew);
    }
}

// Overlap round k found nothing: the overlap loop of this step is done.  The
// flipped list restarts for the edges flipped after this detection.
__device__ __forceinline__ void ovl_check_body(int *ctl, int k, int stamp, const StepBase *base) {
    if (stopped(ctl)) return;
    ctl[K_FL_N] = 0;
    ctl[K_VT_N] = 0;
    ctl[K_FL_EPOCH] = stamp + base->vbase;
    if (ctl_read(ctl, K_TOPO) != 0) {
        ctl[K_REASON] = HALT_TOPOLOGY;
        ctl[K_STAGE] = k;
        ctl[K_HALT] = 1;
        return;
    }
    if (ctl_read(ctl, K_OVL + k) == 0)
        ctl[K_DONE] = 1;
    else
        ctl[K_OVL_ROUNDS] = k + 1;
}

// After the last budgeted round, or where the tail's next one is for many workgroups: overlaps remain after k rounds,
// the host continues.
__device__ __forceinline__ void final_check_body(int *ctl, int k) {
    if (stopped(ctl)) return;
    ctl[K_REASON] = HALT_OVERLAP_BUDGET;
    ctl[K_STAGE] = k;
    ctl[K_HALT] = 1;
}

// Gather: for a queued disk, sum the Jacobi displacement over its star
// (Sec. 2.3 displacement along the unit vector, factor f), starting at the
// neighbour of smallest id so the summation order is independent of flip
// history; truncate the sum to cap_frac * r (Sec. 4.4); reflect at the walls
// (fold into the box when periodic).  One group of lanes per star (star_walk),
// which is recorded for the first evaluation of the repair and the detection
// that follow; the lanes' contributions are added in the canonical order.  The
// time is the chain of the walk: 65,536 disks, 16 us as one thread per star
// walked from one end.

// Displacement of disk v (at pv, radius rv) by its neighbour w; false when they do not overlap.
template <class TP>
__device__ __forceinline__ bool ovl_term(const TP &t, double2 pv, double rv, int w, double2 pw, double f,
                                         double keep, double &cx, double &cy) {
#pragma clang fp contract(off)
    const double dx = sep_p(t, pv.x - pw.x), dy = sep_p(t, pv.y - pw.y);
    const double d = sqrt(dx * dx + dy * dy);
    const double contact = rv + (t.ru > 0.0 ? t.ru : t.rad[w]);
    if (!(d < contact * keep)) return false;
    const double sc = f * (contact - d) / d;
    cx = sc * dx;
    cy = sc * dy;
    return true;
}

// Disk v, queued at idx: its star, and in the group's first lane its position before (pv) and after (np).
template <class TP>
__device__ __forceinline__ Star gather_star(const TP &t, int idx, int v, double f, double cap_frac, double keep,
                                                double2 &pv, double2 &np) {
#pragma clang fp contract(off)
    const int q = star_lane();
    const bool rec = t.tev != nullptr;   // adjoint tape: entry idx of this round for disk idx
    pv = np = t.xy[v];
    const double rv = t.ru > 0.0 ? t.ru : t.rad[v];
    const double L = t.Lr[t.rep_of[v]];
    const Star s = star_walk(t, v);
    if (q == 0) t.star_deg[idx] = s.deg;
    if (s.deg == 0) {
        if (q == 0) {
            t.newpos[idx] = pv;
            topo_err(t);
            atomicAdd(&t.ctl[K_STAR], 1);
        }
        return s;
    }
    const int e = rec ? t.tent_base + t.ctl[K_TAPE_ENT] + idx : 0;
    const bool room = rec && e < t.tcap_ent;
    if (rec && !room && q == 0) atomicOr(&t.ctl[K_TAPE_OVF], 1);
    int na = 0;
    double sx = 0.0, sy = 0.0;
    if (s.deg == kStarLarge) {
        if (q != 0) return s;
        // one lane: the neighbour of smallest id, then the sum around the star from there
        const int h0 = t.vert_he[v];
        int best = h0, bestid = 0x7FFFFFFF, h = h0, guard = 0;
        bool broken = false;
        do {
            const int w = t.he_v[bd_next(h)];
            if (bad_v(t, w)) {
                broken = true;
                break;
            }
            if (w < t.inf && w < bestid) {
                bestid = w;
                best = h;
            }
            h = t.he_twin[bd_prev(h)];
            if (bad_he(t, h) || ++guard > 4096) {
                broken = true;
                break;
            }
        } while (h != h0);
        if (broken) {
            t.newpos[idx] = pv;
            topo_err(t);
            atomicAdd(&t.ctl[K_STAR], 1);
            return s;
        }
        h = best;
        do {
            const int w = t.he_v[bd_next(h)];
            double cx, cy;
            if (w < t.n && ovl_term(t, pv, rv, w, t.xy[w], f, keep, cx, cy)) {
                sx += cx;
                sy += cy;
                if (room && na < MAXACT) t.tenb[(size_t)e * MAXACT + na] = w;
                ++na;
            }
            h = t.he_twin[bd_prev(h)];
        } while (h != best);
    } else {
        const bool two = star_two(s);
        double cx[2], cy[2];
        unsigned hits = 0;   // bit i: neighbour i overlaps
        int bestid = 0x7FFFFFFF, best = 0;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            cx[u] = cy[u] = 0.0;
            if (u == 1 && !two) continue;
            const int i = q + u * kStarLanes;
            bool hit = false;
            if (i < s.deg) {
                t.star[(size_t)idx * kStarMax + i] = s.h[u];
                if (s.w[u] < t.n) hit = ovl_term(t, pv, rv, s.w[u], t.xy[s.w[u]], f, keep, cx[u], cy[u]);
                if (s.w[u] < t.inf && s.w[u] < bestid) {
                    bestid = s.w[u];
                    best = i;
                }
            }
            hits |= (unsigned)((__ballot(hit) >> star_base()) & ((1ull << kStarLanes) - 1ull)) << (u * kStarLanes);
        }
        for (int off = kStarLanes / 2; off > 0; off >>= 1) {
            const int oid = __shfl_xor(bestid, off), ob = __shfl_xor(best, off);
            if (oid < bestid) {
                bestid = oid;
                best = ob;
            }
        }
        // canonical order: neighbours best .. deg - 1, then 0 .. best - 1
        unsigned part = hits & ~((1u << best) - 1u), rest = hits & ((1u << best) - 1u);
        while ((part | rest) != 0) {
            if (part == 0) {
                part = rest;
                rest = 0;
            }
            const int i = __ffs(part) - 1;
            part &= part - 1;
            sx += star_get(cx, i, two);
            sy += star_get(cy, i, two);
            const int w = star_get(s.w, i, two);
            if (room && q == 0 && na < MAXACT) t.tenb[(size_t)e * MAXACT + na] = w;
            ++na;
        }
        if (q != 0) return s;
    }
    if (room) {
        if (na > MAXACT) atomicOr(&t.ctl[K_TAPE_OVF], 2);
        t.tev[e] = v;
        t.tecnt[e] = na < MAXACT ? na : MAXACT;
        t.teold[e] = pv;
        t.tedisp[e] = make_double2(sx, sy);
    }
    const double len = sqrt(sx * sx + sy * sy);
    const double cap = cap_frac * rv;
    if (len > cap) {
        double sc = cap / len;
        sx = sx * sc;
        sy = sy * sc;
        wave_count64(&t.acc[A_CAP_HITS], true);
    }
    const double xv = pv.x, yv = pv.y;
    if (room) {
        t.tewf[2 * (size_t)e] = bd_wall_slope(xv + sx, rv, L);
        t.tewf[2 * (size_t)e + 1] = bd_wall_slope(yv + sy, rv, L);
    }
    np = TP::kPer ? make_double2(bd_wrap(xv + sx, t.P), bd_wrap(yv + sy, t.P))
                   : make_double2(bd_wall(xv + sx, rv, L), bd_wall(yv + sy, rv, L));
    t.newpos[idx] = np;
    return s;
}

template <class TP>
__global__ __launch_bounds__(256) void k_ovl_gather(TP t, int k, double f, double cap_frac, double keep) {
    if (stopped(t.ctl)) return;
    const int ntouched = t.ctl[K_TOUCH + k];
    const int *touched = touched_of(t, k);
    const int i0 = xcd_block() * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    for (int idx = i0 / kStarLanes; idx < ntouched; idx += stride / kStarLanes) {
        double2 pv, np;
        gather_star(t, idx, touched[idx], f, cap_frac, keep, pv, np);
    }
}

__device__ __forceinline__ void move_disk(const Topo &t, int idx, int v, double2 from, double2 to) {
    t.oldpos[idx] = from;
    ((double *)t.x)[v] = to.x;
    ((double *)t.y)[v] = to.y;
    ((double2 *)t.xy)[v] = to;
}

// Adjoint tape: closes the round's entries (written by the gather); one thread.
__device__ __forceinline__ void close_tape_round(const Topo &t, int ntouched) {
    if (t.tev == nullptr) return;
    const int di = t.tdir_base + t.ctl[K_TAPE_DIR];
    if (di < t.tcap_dir)
        t.tdir[di] = make_int2(t.tent_base + t.ctl[K_TAPE_ENT], ntouched);
    else
        atomicOr(&t.ctl[K_TAPE_OVF], 1);
    t.ctl[K_TAPE_ENT] += ntouched;
    t.ctl[K_TAPE_DIR] += 1;
}

__device__ __forceinline__ void ovl_apply_body(const Topo &t, int k, int i0, int stride) {
    if (stopped(t.ctl)) return;
    const int ntouched = t.ctl[K_TOUCH + k];
    if (i0 == 0) close_tape_round(t, ntouched);
    const int *touched = touched_of(t, k);
    for (int idx = i0; idx < ntouched; idx += stride) {
        const int v = touched[idx];
        move_disk(t, idx, v, t.xy[v], t.newpos[idx]);
    }
}

__global__ void k_ovl_apply(Topo t, int k) {
    if (stopped(t.ctl)) return;
    ovl_apply_body(t, k, xcd_block() * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

// The overlap rounds after the first detection in one workgroup, the phases of
// the separate launches with a barrier between them (workgroup-scope
// release/acquire, so every thread sees the previous phase's writes).  Halts
// follow the same rules.  A round is a chain of some twenty dependent steps, so
// what it waits for is latency: of memory, of atomics, and of instructions not
// in the cache.  Small rounds took 13 us with 162 KiB of code (every phase
// inlined for both box kinds), 10 us with 60 KiB; 1,024 disks 64 to 58 us a
// step, 16,001 in the periodic box 272 to 247.
//
// A round of many disks is for many workgroups: the tail takes some 0.11 us a
// disk and round, launches from the host some 120 us a round whatever it moves.
// So a round that queues more than kTailMost disks goes to the host with the
// rest of the step, and more than kTailLong where several rounds before it did
// not bring the number down (kTailFirst).  A step
// from positions where every disk of some patches overlaps, 116 to 137 rounds,
// ms with the 48 rounds the tail holds / so: 2,304 disks 17.2 / 12.6, 5,184 31 /
// 12.7, 14,400 76 / 14.7, 82,944 427 / 18.6, 230,400 1218 / 24; 16,000 disks with
// moves of 0.2 radii 1.80 / 1.24 a step.  With kTailMost 2,048 and 1,024 instead
// of 4,096: 5,000 such disks 1.03 and 1.03 a step for 0.67, 3,000 0.48 and 0.97
// for 0.48.
constexpr int kTailMost = 4096, kTailFirst = 7, kTailLong = 1400;
constexpr int kTailBlock = 1024;

// In one workgroup, after a barrier: true when flip round `slot` has nothing
// left to do, before its evaluation (empty worklist) or after it (no
// candidate).  Leaving the loop there gives the same result as running the
// remaining rounds: without a candidate a round queues only edges whose flip is
// blocked (register_flip), and with positions and topology unchanged those stay
// blocked in every later round.  They exist only beside an inverted triangle (on
// an embedded triangulation the diagonal that a quad must flip to is no edge),
// so the repair ends in HALT_INVALID and the host replays the move, whichever
// round it left at.  The counters were last written by atomics before the
// barrier and are not written again before the decision, so every thread reads
// the same value.
__device__ __forceinline__ bool rounds_done(const Topo &t, int slot, bool evaluated) {
    return ctl_read(t.ctl, (evaluated ? K_CAND : K_WL) + slot) == 0;
}

// Between two phases: true when the step has stopped (the same for every thread).
__device__ __forceinline__ bool tail_sync(const Topo &t) {
    __syncthreads();
    const bool stop = stopped(t.ctl);
    __syncthreads();
    return stop;
}

// Flip rounds [round0, round0 + rounds) of a repair in one workgroup, from
// slot slot0 on.  first_evaluated: the first round's evaluation already ran in
// a launch of many workgroups (the repair after the move scans every edge), so
// it starts with that round's apply; otherwise with the evaluation of the
// worklist in slot0.  The loop ends at the first round with nothing to do.
// Returns true when the step has stopped.
template <class TP>
__device__ __forceinline__ bool repair_rounds_body(const TP &t, int round0, int slot0, int rounds,
                                                   bool first_evaluated) {
    const int i0 = threadIdx.x, stride = blockDim.x;
    if (tail_sync(t)) return true;
    for (int r = 0; r < rounds; ++r) {
        int slot = slot0 + r;
        if (slot >= MAXR) slot -= MAXR;
        const int round = round0 + r;
        if (r > 0 || !first_evaluated) {
            if (rounds_done(t, slot, false)) break;
            flip_eval_list_body<1>(t, round, slot, i0, stride, nullptr);
            if (tail_sync(t)) return true;
        }
        if (rounds_done(t, slot, true)) break;
        flip_apply_body(t, round, slot, i0, stride);
        if (tail_sync(t)) return true;
        flip_fix_body(t, round, slot, i0, stride);
        if (tail_sync(t)) return true;
    }
    return false;
}

// The workgroup keeps the control block in LDS: every phase reads its counts and the stop flags, and every list
// append takes a position there.
__device__ __forceinline__ void ctl_to_lds(Topo &t, int *lds) {
    for (int i = threadIdx.x; i < N_CTL; i += blockDim.x) lds[i] = t.ctl[i];
    __syncthreads();
    t.ctl = lds;
}

template <class TP>
__global__ __launch_bounds__(kTailBlock) void k_repair_rounds(TP t, int round0, int slot0, int rounds,
                                                              int first_evaluated) {
    __shared__ int s_ctl[N_CTL];
    int *ctl = t.ctl;
    ctl_to_lds(t, s_ctl);
    repair_rounds_body(t, round0, slot0, rounds, first_evaluated != 0);
    __syncthreads();
    for (int i = threadIdx.x; i < N_CTL; i += blockDim.x) ctl[i] = s_ctl[i];
}

// Rounds that queue at most one star per group of lanes keep the stars in
// registers: gather, move, then the repair's first evaluation together with the
// tests the detection will make; when no edge flips those tests stand, and the
// round ends without reading a star again.  Each phase has one copy of its code
// (see TopoP).
template <class TP>
__device__ __forceinline__ void tail_body(const TP &t, const TailPlan &p) {
    const int i0 = threadIdx.x, stride = blockDim.x;
    const int g0 = i0 / kStarLanes, gstep = kTailBlock / kStarLanes;
    if (i0 == 0 && t.ctl[K_TOUCH + p.k[0]] > kTailMost) final_check_body(t.ctl, p.k[0]);
    if (tail_sync(t)) return;
    for (int j = 0; j < p.nover; ++j) {
        const int k = p.k[j], knew = p.k[j + 1];
        const int ntouched = t.ctl[K_TOUCH + k];
        const int *touched = touched_of(t, k);
        const bool small = ntouched <= gstep;
        Star s;
        double2 pv, np;
        int r = 0, v = 0, slot = p.slot0[j], round = p.next_round[j], last = slot;
        for (int idx = g0; idx < ntouched; idx += gstep) {
            v = touched[idx];
            s = gather_star(t, idx, v, p.f, p.cap_frac, p.keep, pv, np);
        }
        if (tail_sync(t)) return;
        if (small) {
            if (g0 < ntouched && star_lane() == 0 && s.deg != 0) move_disk(t, g0, v, pv, np);
            if (i0 == 0) close_tape_round(t, ntouched);
        } else {
            ovl_apply_body(t, k, i0, stride);
        }
        if (tail_sync(t)) return;
        bool tested = false;
        for (int idx = g0; idx < ntouched; idx += gstep) {
            if (!small) {
                v = touched[idx];
                s = star_recorded(t, idx);
            }
            StarPos sp;
            tested = eval_star<1>(t, v, s, round + t.base->rbase, slot, sp, nullptr);
            if (small && tested) r = star_test(t, v, s, sp, p.keep);
        }
        const bool none = rounds_done(t, slot, false);   // nothing the repair before left blocked
        if (!none) flip_eval_list_body<1>(t, round, slot, i0, stride, nullptr);
        if (tail_sync(t)) return;
        const bool flips = !rounds_done(t, slot, true);
        for (int rr = 1; flips; ++rr) {   // the repair's rounds, as repair_rounds_body
            flip_apply_body(t, round, slot, i0, stride);
            if (tail_sync(t)) return;
            flip_fix_body(t, round, slot, i0, stride);
            if (tail_sync(t)) return;
            if (rr == p.rounds[j]) break;
            ++round;
            slot = slot + 1 >= MAXR ? 0 : slot + 1;
            last = slot;
            if (rounds_done(t, slot, false)) break;
            flip_eval_list_body<1>(t, round, slot, i0, stride, nullptr);
            if (tail_sync(t)) return;
            if (rounds_done(t, slot, true)) break;
        }
        // this repair's validation with the next round's detection; then the repair's check and the detection's,
        // as the last workgroup of the fused launch does
        int *inv = &t.ctl[K_INV + p.rep[j]];
        const int stamp = p.stamp[j + 1] + t.base->vbase;
        int found = 0;
        for (int idx = g0; idx < ntouched; idx += gstep) {
            if (!small || flips || !tested) {
                v = touched[idx];
                tested = star_after_repair<1>(t, idx, v, inv, p.next_round[j] + t.base->rbase, stamp, p.keep, knew,
                                                  found, nullptr, s, r);
            }
            if (tested) star_commit<1>(t, v, s, r, inv, stamp, knew, found, nullptr);
        }
        found += validate_detect_flipped<1>(t, inv, stamp, p.keep, knew, i0, stride, nullptr);
        wave_sum_add(&t.ctl[K_OVL + knew], found);
        __syncthreads();
        if (i0 == 0) {
            const int next = t.ctl[K_TOUCH + knew];
            repair_check_body(t.ctl, p.rep[j], last);
            ovl_check_body(t.ctl, knew, p.stamp[j + 1], t.base);
            if (j + 1 == p.nover || next > (j < kTailFirst ? kTailMost : kTailLong)) final_check_body(t.ctl, knew);
        }
        if (tail_sync(t)) return;
    }
}

template <class TP>
__global__ __launch_bounds__(kTailBlock) void k_tail(TP t, TailPlan p, StepBase *base, int *ring) {
    __shared__ int s_ctl[N_CTL];
    int *ctl = t.ctl;
    ctl_to_lds(t, s_ctl);
    tail_body(t, p);
    __syncthreads();
    if (p.end) {
        step_end_body(s_ctl, ctl, base, ring, p.r_used, p.v_used);
    } else {
        for (int i = threadIdx.x; i < N_CTL; i += blockDim.x) ctl[i] = s_ctl[i];
    }
}

// Topology snapshot before a repair (skipped once the step has stopped, so the
// snapshot of the failing repair survives).
__global__ void k_snapshot(Topo t, int *snap_v, int *snap_twin, int *snap_vh, int nvh, int vec) {
    if (stopped(t.ctl)) return;
    const int H = 3 * t.T;
    const int H4 = vec ? H / 4 : 0, N4 = vec ? nvh / 4 : 0;   // 16-byte copies when aligned, then the tails
    const int stride = gridDim.x * blockDim.x;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < H4; i += stride) {
        reinterpret_cast<int4 *>(snap_v)[i] = reinterpret_cast<const int4 *>(t.he_v)[i];
        reinterpret_cast<int4 *>(snap_twin)[i] = reinterpret_cast<const int4 *>(t.he_twin)[i];
        if (i < N4) reinterpret_cast<int4 *>(snap_vh)[i] = reinterpret_cast<const int4 *>(t.vert_he)[i];
    }
    for (int i = 4 * H4 + blockIdx.x * blockDim.x + threadIdx.x; i < H; i += stride) {
        snap_v[i] = t.he_v[i];
        snap_twin[i] = t.he_twin[i];
    }
    for (int i = 4 * N4 + blockIdx.x * blockDim.x + threadIdx.x; i < nvh; i += stride) snap_vh[i] = t.vert_he[i];
}

__global__ void k_scatter_oldpos(Topo t, int k, double *xa, double *ya) {
    const int ntouched = t.ctl[K_TOUCH + k];
    const int *touched = touched_of(t, k);
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < ntouched; idx += gridDim.x * blockDim.x) {
        const int v = touched[idx];
        xa[v] = t.oldpos[idx].x;
        ya[v] = t.oldpos[idx].y;
    }
}

// Sub-step i of k of a replayed move from (xa, ya) to (xb, yb); in a periodic
// box (P > 0) along the nearest-image displacement, folded into [0, P).
__global__ void k_interp(int n, int i, int k, const double *xa, const double *ya, const double *xb,
                         const double *yb, double *x, double *y, double2 *xy, double P) {
#pragma clang fp contract(off)
    int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    double nx, ny;
    if (i == k) {
        nx = xb[v];
        ny = yb[v];
    } else if (P > 0.0) {
        const double s = (double)i / (double)k;
        nx = bd_wrap(xa[v] + s * bd_min_image(xb[v] - xa[v], P), P);
        ny = bd_wrap(ya[v] + s * bd_min_image(yb[v] - ya[v], P), P);
    } else {
        const double s = (double)i / (double)k;
        nx = xa[v] + s * (xb[v] - xa[v]);
        ny = ya[v] + s * (yb[v] - ya[v]);
    }
    x[v] = nx;
    y[v] = ny;
    xy[v] = make_double2(nx, ny);
}

inline int grid_for(long items, int cap = kMaxGrid) {
    long b = (items + 255) / 256;
    if (b < 1) b = 1;
    return (int)(b < cap ? b : cap);
}

// Workgroups of the worklist-driven launches: most of them find a short or
// empty list, and an empty launch costs more the more workgroups it has, so
// the grid grows with the problem (lists grow with it), from 16 to 128.
inline int list_grid(const Sim &s) {
    const int g = s.n / 1024;
    return g < 16 ? 16 : (g > kListGridMax ? kListGridMax : g);
}

// Workgroups of the launches with one group of lanes per star.
inline int star_grid(const Sim &s) { return std::min(kStarGridMax, list_grid(s) * 8); }

// Calls f with the topology typed by the box kind.
template <class F>
void with_box(const Topo &t, F &&f) {
    if (t.P > 0.0) {
        TopoP<true> tp;
        static_cast<Topo &>(tp) = t;
        f(tp);
    } else {
        TopoP<false> tp;
        static_cast<Topo &>(tp) = t;
        f(tp);
    }
}

}  // namespace

void launch_flip_eval_full(Sim &s, int round, int slot, int reversal, bool snapshot) {
    round -= s.rbase;
    const Topo t = topo_of(s);
    const Snapshot snap = snapshot ? Snapshot{s.snap_v, s.snap_twin, s.snap_vh, s.nv + s.R} : Snapshot{};
    with_box(t, [&](auto tp) {
        const int grid = grid_for((long)(s.T + 3) / 4 * 1024 / kEvalBlock, kEvalGrid);
        hipLaunchKernelGGL(k_flip_eval_full<decltype(tp)>, dim3(grid), dim3(kEvalBlock), 0, s.stream, tp, round, slot,
                           reversal, snap);
    });
}

void launch_flip_eval_list(Sim &s, int round, int slot) {
    round -= s.rbase;
    const Topo t = topo_of(s);
    with_box(t, [&](auto tp) {
        hipLaunchKernelGGL(k_flip_eval_list<decltype(tp)>, dim3(list_grid(s)), dim3(256), 0, s.stream, tp, round, slot);
    });
}

void launch_flip_eval_star(Sim &s, int k, int round, int slot) {
    round -= s.rbase;
    const Topo t = topo_of(s);
    with_box(t, [&](auto tp) {
        hipLaunchKernelGGL(k_flip_eval_star<decltype(tp)>, dim3(star_grid(s)), dim3(256), 0, s.stream, tp, k, round,
                           slot);
    });
}

void launch_flip_apply(Sim &s, int round, int slot) {
    round -= s.rbase;
    const Topo t = topo_of(s);
    hipLaunchKernelGGL(k_flip_apply, dim3(list_grid(s)), dim3(256), 0, s.stream, t, round, slot);
}

void launch_flip_fix(Sim &s, int round, int slot) {
    round -= s.rbase;
    const Topo t = topo_of(s);
    hipLaunchKernelGGL(k_flip_fix, dim3(list_grid(s)), dim3(256), 0, s.stream, t, round, slot);
}

void launch_validate(Sim &s, int rep) {
    const Topo t = topo_of(s);
    with_box(t, [&](auto tp) {
        hipLaunchKernelGGL(k_validate<decltype(tp)>, dim3(grid_for((s.T + 3) / 4)), dim3(kScanBlock), 0, s.stream, tp,
                           rep);
    });
}

void launch_ovl_detect(Sim &s, int vstamp, int k, int check, int vrep, int vlast) {
    vstamp -= s.vbase;
    const Topo t = topo_of(s);
    with_box(t, [&](auto tp) {
        hipLaunchKernelGGL(k_ovl_detect<decltype(tp)>, dim3(grid_for((s.T + 3) / 4)), dim3(kDetBlock), 0, s.stream, tp,
                           vstamp, 1.0 - s.p.contact_tol, k, check, vrep, vlast);
    });
}

void launch_validate_detect_local(Sim &s, int rep, int k, int rfirst, int last, int vstamp, int knew, int check) {
    vstamp -= s.vbase;
    rfirst -= s.rbase;
    const Topo t = topo_of(s);
    with_box(t, [&](auto tp) {
        hipLaunchKernelGGL(k_validate_detect_local<decltype(tp)>, dim3(star_grid(s)), dim3(256), 0, s.stream, tp, rep,
                           k, rfirst, last, vstamp, 1.0 - s.p.contact_tol, knew, check);
    });
}

void launch_ovl_gather(Sim &s, int k) {
    const Topo t = topo_of(s);
    with_box(t, [&](auto tp) {
        hipLaunchKernelGGL(k_ovl_gather<decltype(tp)>, dim3(star_grid(s)), dim3(256), 0, s.stream, tp, k,
                           s.p.overlap_factor, s.p.cap_frac, 1.0 - s.p.contact_tol);
    });
}

void launch_ovl_apply(Sim &s, int k) {
    const Topo t = topo_of(s);
    hipLaunchKernelGGL(k_ovl_apply, dim3(list_grid(s)), dim3(256), 0, s.stream, t, k);
}

void launch_tail(Sim &s, const TailPlan &plan) {
    const Topo t = topo_of(s);
    with_box(t, [&](auto tp) {
        hipLaunchKernelGGL(k_tail<decltype(tp)>, dim3(1), dim3(kTailBlock), 0, s.stream, tp, plan, s.dbase, s.ring);
    });
}

void launch_repair_rounds(Sim &s, int round0, int slot0, int rounds, bool first_evaluated) {
    const Topo t = topo_of(s);
    with_box(t, [&](auto tp) {
        hipLaunchKernelGGL(k_repair_rounds<decltype(tp)>, dim3(1), dim3(kTailBlock), 0, s.stream, tp, round0 - s.rbase,
                           slot0, rounds, first_evaluated ? 1 : 0);
    });
}

void launch_snapshot(Sim &s) {
    const Topo t = topo_of(s);
    const void *p[] = {s.he_v, s.he_twin, s.vert_he, s.snap_v, s.snap_twin, s.snap_vh};
    int vec = 1;
    for (const void *q : p) vec &= ((uintptr_t)q % 16 == 0) ? 1 : 0;
    hipLaunchKernelGGL(k_snapshot, dim3(grid_for(s.H / 4, kScanGrid)), dim3(256), 0, s.stream, t, s.snap_v,
                       s.snap_twin, s.snap_vh, s.nv + s.R, vec);
}

void launch_scatter_oldpos(Sim &s, int k) {
    const Topo t = topo_of(s);
    hipLaunchKernelGGL(k_scatter_oldpos, dim3(grid_for(s.n)), dim3(256), 0, s.stream, t, k, s.xa, s.ya);
}

void launch_interp(Sim &s, int i, int k) {
    hipLaunchKernelGGL(k_interp, dim3((s.n + 255) / 256), dim3(256), 0, s.stream, s.n, i, k, s.xa, s.ya, s.xb,
                       s.yb, s.x, s.y, s.xy, s.period);
}

}  // namespace bd
