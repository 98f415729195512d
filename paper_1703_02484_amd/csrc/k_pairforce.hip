// Stateless pair forces of the Sec. 2.2 law on caller device arrays:
//   F_i = sum_{j != i} K[s_i][s_j] g(d_ij) (r_i - r_j) / d_ij
// for positions and species that live in device memory owned by the caller,
// with no simulation handle.
//
// Four layouts, chosen from n, the precision, the law and whether there is a
// cutoff (pf_plan); all but cells are bound by the VALU:
//   rows   (few particles) one wavefront per particle i, its lanes over the
//          j; the 64 partial sums are added across the wavefront in FP64.  One launch, no working memory: with few
//          particles the time is the launch and the chain of one lane's j.
//   tiles  the j range is cut into J equal splits; one workgroup takes
//          256 * P particles i (P per lane) against one split, staged through
//          LDS in blocks of kPfJ (the shared-memory broadcast of the paper's
//          n-body kernel, Sec. 6: every lane reads the same j from LDS).  A
//          staged block is ordered by species, so the strength matrix leaves
//          the pair loop: it weights the sum over each species' part of the
//          block.  part[split][i] holds the weighted sums; a second kernel
//          adds the J splits in FP64 in split order.
//   sym    (inverse square, no cutoff, larger n) the particles are sorted by
//          species and every pair of chunks of them is taken once, both sides
//          from one evaluation.
//   cells  (a cutoff) the particles are put into square cells of the cutoff's
//          side and each is taken against its 3 x 3 cells: launches of a few
//          us each instead of n^2 distance tests.  Positions it cannot bin, and
//          ones so crowded that most pairs would be tested anyway, go to the
//          tiles, which are launched behind it and do nothing otherwise.
// None depends on the launch timing.  The only device memory beyond the
// caller's inputs and outputs is `part` (J * n * 2 values of the working
// precision), the sorted particles and chunk sums of sym, or the cells' arrays.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "../../include/bd.h"

namespace {

constexpr int kPfBlock = 256;
constexpr int kPfJ = 512;                      // j staged in LDS per pass
constexpr int kPfTargetGroups = 2048;          // workgroups aimed for (8 per CU)
constexpr int kPfMaxSplits = 64;
constexpr int kPfChunks = kPfJ / 64;           // wavefront-sized pieces of a staged block

struct PfLaw {
    int kind, S;
    double q, A, lam, cutoff;
    double K[BD_MAX_SPECIES * BD_MAX_SPECIES];
};

template <typename T>
struct Vec2;
template <>
struct Vec2<float> {
    using type = float2;
};
template <>
struct Vec2<double> {
    using type = double2;
};

// The law's form, fixed at compile time: the inverse-square law r / r^3, any other power, the screened law.
enum { PF_Q2 = 0, PF_POWER = 1, PF_SCREENED = 2 };

template <typename T>
struct PfConst {
    T cut2, expo, invlam, A;
    __device__ explicit PfConst(const PfLaw &law)
        : cut2(law.cutoff > 0.0 ? (T)(law.cutoff * law.cutoff) : (T)0), expo((T)(-0.5 * (law.q + 1.0))),
          invlam((T)(1.0 / law.lam)), A((T)law.A) {}
};

// g(d)/d for the law (the factor multiplying r_i - r_j).  Inverse square: d^-3 from the hardware estimate of
// d2^-1/2; in FP64 corrected by y^3 (1 + 3/2 e + 15/8 e^2), e = 1 - d2 y^2, which leaves an error of order
// e^3 (below rounding).  d2 is capped where d^-3 is 0 anyway, so that an overflowed d2 gives 0 and not NaN.
template <int LAW>
__device__ __forceinline__ float law_factor(float d2, const PfConst<float> &c) {
    if (LAW == PF_Q2) {
        const float r = __builtin_amdgcn_rsqf(d2);
        return r * r * r;
    }
    if (LAW == PF_POWER) return powf(d2, c.expo);
    const float d = sqrtf(d2);
    return c.A * expf(-d * c.invlam) / d2;
}
template <int LAW>
__device__ __forceinline__ double law_factor(double d2, const PfConst<double> &c) {
    if (LAW == PF_Q2) {
        d2 = fmin(d2, 1e300);
        const double y = __builtin_amdgcn_rsq(d2);
        const double y2 = y * y;
        const double e = fma(-d2, y2, 1.0);
        return (y2 * y) * fma(fma(1.875, e, 1.5), e, 1.0);
    }
    if (LAW == PF_POWER) return pow(d2, c.expo);
    const double d = sqrt(d2);
    return c.A * exp(-d * c.invlam) / d2;
}

// ---------------------------------------------------------------- rows
// Sum over the wavefront in a fixed order; every lane ends with it.
__device__ __forceinline__ double wave_sum(double v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// One wavefront per particle i, lanes over j.  The piece of 64 j that holds i, and the ragged last one, test each
// j; the others do not.  777 particles in FP64: 8 us (4 workgroups that each took 512 particles: 178 us).
template <typename T, int LAW, bool CUT>
__global__ __launch_bounds__(kPfBlock) void k_pf_rows(int n, const double *__restrict__ xy,
                                                      const int32_t *__restrict__ species, PfLaw law,
                                                      double *__restrict__ f) {
    __shared__ T kw[BD_MAX_SPECIES * BD_MAX_SPECIES];
    const int S = law.S;
    for (int k = threadIdx.x; k < S * S; k += kPfBlock) kw[k] = (T)law.K[k];
    __syncthreads();
    const PfConst<T> c(law);
    const int lane = threadIdx.x & 63;
    const int i = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kPfBlock / 64) + (threadIdx.x >> 6)));
    if (i >= n) return;   // after the workgroup's only barrier
    const T xi = (T)xy[2 * (size_t)i], yi = (T)xy[2 * (size_t)i + 1];
    const int si = species[i] * S;
    T ax = (T)0, ay = (T)0;
    auto piece = [&](int b, auto check) {
        constexpr bool CHECK = decltype(check)::value;
        const int j = b * 64 + lane;
        const int jc = CHECK ? min(j, n - 1) : j;
        const T xj = (T)xy[2 * (size_t)jc], yj = (T)xy[2 * (size_t)jc + 1];
        const int sj = S > 1 ? species[jc] : 0;
        const T dx = xi - xj, dy = yi - yj;
        const T d2 = dx * dx + dy * dy;
        T g = law_factor<LAW>(d2, c);
        if (S > 1) g *= kw[si + sj];
        if (CUT) g = d2 > c.cut2 ? (T)0 : g;
        if (CHECK) g = (j >= n || j == i) ? (T)0 : g;
        ax += dx * g;
        ay += dy * g;
    };
    using Yes = std::integral_constant<bool, true>;
    using No = std::integral_constant<bool, false>;
    const int own = i >> 6, nfull = n >> 6;
    const int a = min(own, nfull);
#pragma unroll 4
    for (int b = 0; b < a; ++b) piece(b, No{});
    if (own < nfull) piece(own, Yes{});
#pragma unroll 4
    for (int b = own + 1; b < nfull; ++b) piece(b, No{});
    if (nfull * 64 < n) piece(nfull, Yes{});
    double fx = wave_sum((double)ax), fy = wave_sum((double)ay);
    if (S == 1) {
        fx *= (double)kw[0];
        fy *= (double)kw[0];
    }
    if (lane == 0) {
        f[2 * (size_t)i] = fx;
        f[2 * (size_t)i + 1] = fy;
    }
}

// ---------------------------------------------------------------- tiles
// A block of j staged in LDS, ordered by species (ascending j inside a species): seg[s] .. seg[s + 1) holds species s.
template <typename T>
struct PfStage {
    typename Vec2<T>::type pos[kPfJ];
    short idx[kPfJ];                                  // j - jb
    int cnt[BD_MAX_SPECIES * kPfChunks];              // per species and wavefront-sized piece: count, then start
    int seg[BD_MAX_SPECIES + 1];
};

template <typename T>
__device__ __forceinline__ void pf_stage(PfStage<T> &st, int S, int jb, int m, const double *__restrict__ xy,
                                         const int32_t *__restrict__ species) {
    using T2 = typename Vec2<T>::type;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int kRounds = kPfJ / kPfBlock;
    __syncthreads();   // the previous block has been read
    if (S == 1) {
        for (int k = tid; k < m; k += kPfBlock) {
            T2 v;
            v.x = (T)xy[2 * (size_t)(jb + k)];
            v.y = (T)xy[2 * (size_t)(jb + k) + 1];
            st.pos[k] = v;
            st.idx[k] = (short)k;
        }
        if (tid == 0) {
            st.seg[0] = 0;
            st.seg[1] = m;
        }
        __syncthreads();
        return;
    }
    T2 v[kRounds];
    int sp[kRounds], rank[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int k = r * kPfBlock + tid;
        sp[r] = k < m ? species[jb + k] : -1;
        if (k < m) {
            v[r].x = (T)xy[2 * (size_t)(jb + k)];
            v[r].y = (T)xy[2 * (size_t)(jb + k) + 1];
        }
        for (int s = 0; s < S; ++s) {
            const unsigned long long mm = __ballot(sp[r] == s);
            if (sp[r] == s) rank[r] = __popcll(mm & ((1ull << lane) - 1ull));
            if (lane == 0) st.cnt[s * kPfChunks + r * (kPfBlock / 64) + wave] = __popcll(mm);
        }
    }
    __syncthreads();
    if (tid < 64) {   // exclusive scan of the S * kPfChunks <= 64 counts, species by species
        const int c = tid < S * kPfChunks ? st.cnt[tid] : 0;
        int incl = c;
        for (int off = 1; off < 64; off <<= 1) {
            const int u = __shfl_up(incl, off);
            if (tid >= off) incl += u;
        }
        if (tid < S * kPfChunks) st.cnt[tid] = incl - c;
        if (tid < S * kPfChunks && tid % kPfChunks == 0) st.seg[tid / kPfChunks] = incl - c;
        if (tid == S * kPfChunks - 1) st.seg[S] = incl;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int s = sp[r];
        if ((unsigned)s >= (unsigned)S) continue;
        const int at = st.cnt[s * kPfChunks + r * (kPfBlock / 64) + wave] + rank[r];
        st.pos[at] = v[r];
        st.idx[at] = (short)(r * kPfBlock + tid);
    }
    __syncthreads();
}

// Adds the staged j [k0, k1) to the sums of P particles i.  SELF: the block may hold i itself (at index own[p]).  CUT:
// pairs beyond the cutoff add 0.
template <typename T, int LAW, int P, bool SELF, bool CUT>
__device__ __forceinline__ void pf_block(const PfStage<T> &st, int k0, int k1, const PfConst<T> &c, const T (&xi)[P],
                                         const T (&yi)[P], const int (&own)[P], T (&ax)[P], T (&ay)[P]) {
#pragma unroll 4
    for (int k = k0; k < k1; ++k) {
        const auto q = st.pos[k];
        const int jk = SELF ? (int)st.idx[k] : 0;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const T dx = xi[p] - q.x, dy = yi[p] - q.y;
            const T d2 = dx * dx + dy * dy;
            T g = law_factor<LAW>(d2, c);
            if (SELF) g = own[p] == jk ? (T)0 : g;
            if (CUT) g = d2 > c.cut2 ? (T)0 : g;
            ax[p] += dx * g;
            ay[p] += dy * g;
        }
    }
}

// The same for blocks most of whose pairs are beyond the cutoff.  A law costs many times the test, so a lane only notes
// the staged j inside its cutoff (kPfHits per particle at most) and the wavefront evaluates the noted pairs together,
// when a lane's list is full and at the end of the part: each lane still adds its pairs in staged order.
constexpr int kPfHits = 16;

template <typename T, int LAW, int P, bool SELF>
__device__ __forceinline__ void pf_block_cut(const PfStage<T> &st, short (&hit)[P][kPfHits][kPfBlock], int k0, int k1,
                                             const PfConst<T> &c, const T (&xi)[P], const T (&yi)[P],
                                             const int (&own)[P], T (&ax)[P], T (&ay)[P]) {
    const int tid = threadIdx.x;
    int cnt[P];
#pragma unroll
    for (int p = 0; p < P; ++p) cnt[p] = 0;
    auto evaluate = [&](int p, T &sx, T &sy) {
        for (int h = 0; __ballot(h < cnt[p]) != 0; ++h) {
            if (h < cnt[p]) {
                const auto q = st.pos[hit[p][h][tid]];
                const T dx = xi[p] - q.x, dy = yi[p] - q.y;
                const T g = law_factor<LAW>(dx * dx + dy * dy, c);
                sx += dx * g;
                sy += dy * g;
            }
        }
        cnt[p] = 0;
    };
    auto test = [&](int k, const typename Vec2<T>::type &q, int jk) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const T dx = xi[p] - q.x, dy = yi[p] - q.y;
            const T d2 = dx * dx + dy * dy;
            bool in = !(d2 > c.cut2);   // a d2 that is not a number is evaluated
            if (SELF) in = in && own[p] != jk;
            if (__ballot(in) != 0) {
                if (in) hit[p][cnt[p]++][tid] = (short)k;
                if (__ballot(cnt[p] == kPfHits) != 0) evaluate(p, ax[p], ay[p]);
            }
        }
    };
    constexpr int kU = 4;   // staged j read ahead
    int k = k0;
    for (; k + kU <= k1; k += kU) {
        typename Vec2<T>::type q[kU];
        int jk[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            q[u] = st.pos[k + u];
            jk[u] = SELF ? (int)st.idx[k + u] : 0;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) test(k + u, q[u], jk[u]);
    }
    for (; k < k1; ++k) test(k, st.pos[k], SELF ? (int)st.idx[k] : 0);
#pragma unroll
    for (int p = 0; p < P; ++p) evaluate(p, ax[p], ay[p]);
}

// Pairs of the wavefront inside the cutoff, of its 64 P kPfProbe with kPfProbe of the block's m staged j.
constexpr int kPfProbe = 8;

template <typename T, int P>
__device__ __forceinline__ int pf_inside(const PfStage<T> &st, int m, const PfConst<T> &c, const T (&xi)[P],
                                         const T (&yi)[P]) {
    int inside = 0;
#pragma unroll
    for (int u = 0; u < kPfProbe; ++u) {
        const auto q = st.pos[u * m / kPfProbe];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const T dx = xi[p] - q.x, dy = yi[p] - q.y;
            inside += __popcll(__ballot(!(dx * dx + dy * dy > c.cut2)));
        }
    }
    return inside;
}

// VALU-bound.  110,000 particles, FP32 inverse square, no cutoff: 2.9 ms, 9 instructions an ordered pair at 0.96 of the
// issue rate (11.8 ms with the strength and the self test in the pair loop and an IEEE square root and division).
// Screened law, FP64, 110,000: without a cutoff 22.8 ms (29.5), cutoff 0.3 of the box 15.4 (29.3, the law evaluated
// wherever one of the wavefront's lanes was in range), beyond the box 23.8 (29.6; 32.1 noting every pair).  That law in
// FP64 with a cutoff is held to 128 registers for four wavefronts a SIMD: 129 and three cost 7 %.
// grid (ceil(n / (256 P)), J); part[split * n + i] = sum over the split's j of K[s_i][s_j] g (r_i - r_j) / d.
template <typename T, int LAW, bool CUT, int P>
__global__ __launch_bounds__(kPfBlock, sizeof(T) == 8 && LAW == PF_SCREENED && CUT ? 4 : 1) void k_pf_tiles(
    int n, int J, const double *__restrict__ xy, const int32_t *__restrict__ species, PfLaw law,
    typename Vec2<T>::type *__restrict__ part, const int *__restrict__ crowded) {
    using T2 = typename Vec2<T>::type;
    __shared__ PfStage<T> st;
    if (crowded && !*crowded) return;   // the cells have done it
    __shared__ T kw[BD_MAX_SPECIES * BD_MAX_SPECIES];
    __shared__ short hit[CUT ? P : 1][CUT ? kPfHits : 1][CUT ? kPfBlock : 1];
    const int S = law.S;
    for (int k = threadIdx.x; k < S * S; k += kPfBlock) kw[k] = (T)law.K[k];   // read after pf_stage's barriers
    const PfConst<T> c(law);
    const int ib = blockIdx.x * kPfBlock * P;
    T xi[P], yi[P], fx[P], fy[P];
    int ii[P], si[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int i = ib + p * kPfBlock + threadIdx.x;
        const int ic = i < n ? i : n - 1;
        ii[p] = i;
        xi[p] = (T)xy[2 * (size_t)ic];
        yi[p] = (T)xy[2 * (size_t)ic + 1];
        si[p] = species[ic] * S;
        fx[p] = (T)0;
        fy[p] = (T)0;
    }
    // with a cutoff the pairs beyond it are skipped: a coordinate at infinity, whose pairs all lie beyond it but give
    // 0 * inf, is found here instead (0 * x is 0 for every finite x)
    __shared__ int at_infinity, inside[2];
    int turn = 0;
    T zx = (T)0, zy = (T)0;
    if (CUT && threadIdx.x == 0) at_infinity = inside[0] = 0;   // read after pf_stage's barriers
    const long long per = ((long long)n + J - 1) / J;
    const int j0 = (int)min((long long)n, per * blockIdx.y);
    const int j1 = (int)min((long long)n, per * (blockIdx.y + 1));
    for (int jb = j0; jb < j1; jb += kPfJ) {
        const int m = min(kPfJ, j1 - jb);
        pf_stage<T>(st, S, jb, m, xy, species);
        if (CUT)
            for (int k = threadIdx.x; k < m; k += kPfBlock) {
                zx += (T)0 * (T)xy[2 * (size_t)(jb + k)];
                zy += (T)0 * (T)xy[2 * (size_t)(jb + k) + 1];
            }
        const bool self = jb < ib + kPfBlock * P && jb + m > ib;   // uniform in the workgroup
        int own[P];
#pragma unroll
        for (int p = 0; p < P; ++p) own[p] = ii[p] - jb;
        // Noting pays where less than kLine / 64 of the pairs are inside.  40,001 particles, us noting with a share of
        // 0.23 and of 0.48 / pair by pair: screened FP32 1217, 2070 / 1940, FP64 2190, 3851 / 3400; q = 6 FP32 2698,
        // 5176 / 5500, FP64 4813, 9259 / 9350; inverse square FP64 1114, 1605 / 1080, FP32 804, 1094 / 640 (never).
        // The wavefronts wait for one another at the next block, so they decide together.
        constexpr int kLine = !CUT ? 0 : LAW == PF_POWER ? 33 : LAW == PF_SCREENED ? 27 : sizeof(T) == 8 ? 20 : 0;
        bool note = false;
        if (kLine > 0) {
            const int in = pf_inside<T, P>(st, m, c, xi, yi);
            if ((threadIdx.x & 63) == 0) atomicAdd(&inside[turn], in);
            __syncthreads();
            note = inside[turn] < kLine * P * kPfProbe * (kPfBlock / 64);
            turn ^= 1;   // the other one was read before the last block was staged
            if (threadIdx.x == 0) inside[turn] = 0;
        }
        for (int s = 0; s < S; ++s) {
            const int k0 = __builtin_amdgcn_readfirstlane(st.seg[s]);
            const int k1 = __builtin_amdgcn_readfirstlane(st.seg[s + 1]);
            T ax[P], ay[P];
#pragma unroll
            for (int p = 0; p < P; ++p) ax[p] = ay[p] = (T)0;
            if (note) {
                if constexpr (CUT) {
                    if (self)
                        pf_block_cut<T, LAW, P, true>(st, hit, k0, k1, c, xi, yi, own, ax, ay);
                    else
                        pf_block_cut<T, LAW, P, false>(st, hit, k0, k1, c, xi, yi, own, ax, ay);
                }
            } else if (self) {
                pf_block<T, LAW, P, true, CUT>(st, k0, k1, c, xi, yi, own, ax, ay);
            } else {
                pf_block<T, LAW, P, false, CUT>(st, k0, k1, c, xi, yi, own, ax, ay);
            }
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const T w = kw[si[p] + s];
                fx[p] += w * ax[p];
                fy[p] += w * ay[p];
            }
        }
    }
    if (CUT) {
        if (zx != (T)0) atomicOr(&at_infinity, 1);
        if (zy != (T)0) atomicOr(&at_infinity, 2);
        __syncthreads();
        const T nan = (T)NAN;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            fx[p] += (at_infinity & 1) ? nan : (T)0 * xi[p];
            fy[p] += (at_infinity & 2) ? nan : (T)0 * yi[p];
        }
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        if (ii[p] < n) {
            T2 v;
            v.x = fx[p];
            v.y = fy[p];
            part[(size_t)blockIdx.y * n + ii[p]] = v;
        }
    }
}

// f[2i], f[2i+1] = sum over the splits in split order, in FP64.
template <typename T>
__global__ void k_pf_reduce(int n, int J, const typename Vec2<T>::type *__restrict__ part, double *__restrict__ f,
                            const int *__restrict__ crowded) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || (crowded && !*crowded)) return;
    double fx = 0.0, fy = 0.0;
#pragma unroll 8
    for (int s = 0; s < J; ++s) {
        const auto v = part[(size_t)s * n + i];
        fx += (double)v.x;
        fy += (double)v.y;
    }
    f[2 * (size_t)i] = fx;
    f[2 * (size_t)i + 1] = fy;
}

// ---------------------------------------------------------------- sym
// Particles sorted by species (ascending index inside one), in chunks of at most C of one species (a species' range cut
// into equal parts).  part[c * n + k]: the sum of sorted particle k over chunk c, without the strength.
template <typename T>
struct PfSym {
    using T2 = typename Vec2<T>::type;
    int *count;    // [blocks of kSortBlock][BD_MAX_SPECIES] particles of each species
    int *total;    // [BD_MAX_SPECIES]
    int *sid;      // [n] particle at each place
    T2 *pos;       // [n]
    T2 *part;      // [rows][n]
};

constexpr int kSortBlock = 1024;

// Counts of a block's species, wave by wave: in LDS for the block's own places, summed in `count` for the others.
__device__ __forceinline__ int pf_wave_count(int s, int S, int (*wcnt)[BD_MAX_SPECIES]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int rank = 0;
    for (int b = 0; b < S; ++b) {
        const unsigned long long m = __ballot(s == b);
        if (s == b) rank = __popcll(m & ((1ull << lane) - 1ull));
        if (lane == 0) wcnt[wave][b] = __popcll(m);
    }
    __syncthreads();
    return rank;
}

__global__ __launch_bounds__(kSortBlock) void k_pf_count(int n, int S, const int32_t *__restrict__ species,
                                                         int *__restrict__ count) {
    __shared__ int wcnt[kSortBlock / 64][BD_MAX_SPECIES];
    const int i = blockIdx.x * kSortBlock + threadIdx.x;
    pf_wave_count(i < n ? species[i] : -1, S, wcnt);
    if (threadIdx.x < S) {
        int c = 0;
        for (int w = 0; w < kSortBlock / 64; ++w) c += wcnt[w][threadIdx.x];
        count[blockIdx.x * BD_MAX_SPECIES + threadIdx.x] = c;
    }
}

template <typename T>
__global__ __launch_bounds__(kSortBlock) void k_pf_sort(int n, int S, const double *__restrict__ xy,
                                                        const int32_t *__restrict__ species, PfSym<T> a) {
    __shared__ int wcnt[kSortBlock / 64][BD_MAX_SPECIES];
    __shared__ int before[BD_MAX_SPECIES], total[BD_MAX_SPECIES];
    if (threadIdx.x < BD_MAX_SPECIES) before[threadIdx.x] = total[threadIdx.x] = 0;
    const int i = blockIdx.x * kSortBlock + threadIdx.x;
    const int s = i < n ? species[i] : -1;
    const int rank = pf_wave_count(s, S, wcnt);
    for (int k = threadIdx.x; k < (int)gridDim.x * BD_MAX_SPECIES; k += kSortBlock) {
        const int b = k % BD_MAX_SPECIES;
        if (b >= S) continue;
        const int c = a.count[k];
        atomicAdd(&total[b], c);
        if (k / BD_MAX_SPECIES < (int)blockIdx.x) atomicAdd(&before[b], c);
    }
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x < BD_MAX_SPECIES) a.total[threadIdx.x] = total[threadIdx.x];
    if ((unsigned)s >= (unsigned)S) return;
    int at = before[s] + rank;
    for (int b = 0; b < s; ++b) at += total[b];
    for (int w = 0; w < (int)threadIdx.x >> 6; ++w) at += wcnt[w][s];
    typename Vec2<T>::type v;
    v.x = (T)xy[2 * (size_t)i];
    v.y = (T)xy[2 * (size_t)i + 1];
    a.pos[at] = v;
    a.sid[at] = i;
}

// Number of chunks, and the range and species of chunk c.
__device__ __forceinline__ int pf_chunks(const int *total, int S, int C) {
    int nc = 0;
    for (int b = 0; b < S; ++b) nc += (total[b] + C - 1) / C;
    return nc;
}
__device__ __forceinline__ int pf_chunk(const int *total, int S, int C, int c, int &k0, int &k1) {
    int base = 0;
    for (int b = 0; b < S; ++b) {
        const int m = total[b], nb = (m + C - 1) / C;
        if (c < nb) {
            k0 = base + (int)((long long)m * c / nb);
            k1 = base + (int)((long long)m * (c + 1) / nb);
            return b;
        }
        c -= nb;
        base += m;
    }
    k0 = k1 = 0;
    return 0;
}

template <typename T>
__device__ __forceinline__ T pf_rot(T v) {   // lane l takes lane l + 1's value
    if constexpr (sizeof(T) == 4) {
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x134, 0xF, 0xF, true));
    } else {
        const long long b = __double_as_longlong(v);
        const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffll), 0x134, 0xF, 0xF, true);
        const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x134, 0xF, 0xF, true);
        return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
    }
}

// 64 steps of a group of 64 Q particles j, Q per lane, turning around the wavefront with their sums.  SELF: the chunk
// with itself, where at step 0 place p of the lane meets itself in place p - same of the group.  PAD: places past the
// chunk's end (lane + 64 p >= ni, j >= nj) do not act.
template <typename T, int P, int Q, bool SELF, bool PAD>
__device__ __forceinline__ void pf_sym_group(const PfConst<T> &c, const T (&xi)[P], const T (&yi)[P], T (&fx)[P],
                                             T (&fy)[P], T (&xj)[Q], T (&yj)[Q], T (&gx)[Q], T (&gy)[Q], int same,
                                             int ni, int nj) {
    const int lane = threadIdx.x & 63;
    for (int t = 0; t < 64; ++t) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const T dx = xi[p] - xj[q], dy = yi[p] - yj[q];
                T g = law_factor<PF_Q2>(dx * dx + dy * dy, c);
                if (SELF) g = t == 0 && p - same == q ? (T)0 : g;
                if (PAD) g = p * 64 + lane < ni && q * 64 + ((lane + t) & 63) < nj ? g : (T)0;
                const T ex = dx * g, ey = dy * g;
                fx[p] += ex;
                fy[p] += ey;
                gx[q] -= ex;
                gy[q] -= ey;
            }
            xj[q] = pf_rot(xj[q]);
            yj[q] = pf_rot(yj[q]);
            gx[q] = pf_rot(gx[q]);
            gy[q] = pf_rot(gy[q]);
        }
    }
}

// One pair of chunks A <= B per workgroup of W wavefronts: the wavefront's 64 P particles of A in registers, those of B
// in groups that the wavefronts take staggered, adding a group's sums to one LDS copy in a fixed order.
// VALU-bound, per unordered pair 11 instructions and 4 / P moves in FP32 against 2 x 9 with both orders: 65,536
// particles, the whole call 0.75 ms (sort and reduction 0.02 of it), 0.96 with both orders.
template <typename T, int P, int W, int Q>
__global__ __launch_bounds__(64 * W) void k_pf_sym(int n, PfLaw law, PfSym<T> a) {
    using T2 = typename Vec2<T>::type;
    constexpr int C = 64 * P * W;
    __shared__ T2 jsum[C];
    const int nc = pf_chunks(a.total, law.S, C);
    const int tile = blockIdx.x;
    if ((long long)tile >= (long long)nc * (nc + 1) / 2) return;   // uniform in the workgroup
    int cb = (int)((sqrt(8.0 * tile + 1.0) - 1.0) * 0.5);
    while ((long long)cb * (cb + 1) / 2 > tile) --cb;
    while ((long long)(cb + 1) * (cb + 2) / 2 <= tile) ++cb;
    int ca = tile - (int)((long long)cb * (cb + 1) / 2);
    int i0, i1, j0, j1;
    pf_chunk(a.total, law.S, C, ca, i0, i1);
    pf_chunk(a.total, law.S, C, cb, j0, j1);
    if (i1 - i0 < j1 - j0) {   // the longer one in registers: the time is the number of groups of the other
        auto swap = [](int &x, int &y) {
            const int z = x;
            x = y;
            y = z;
        };
        swap(ca, cb);
        swap(i0, j0);
        swap(i1, j1);
    }
    const bool self = ca == cb;
    const PfConst<T> c(law);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int ni = i1 - i0, nj = j1 - j0, iw = wave * 64 * P;
    T xi[P], yi[P], fx[P], fy[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int k = iw + p * 64 + lane;
        const T2 v = a.pos[i0 + (k < ni ? k : 0)];
        xi[p] = v.x;
        yi[p] = v.y;
        fx[p] = fy[p] = (T)0;
    }
    if (!self)
        for (int k = threadIdx.x; k < nj; k += 64 * W) {
            T2 z;
            z.x = z.y = (T)0;
            jsum[k] = z;
        }
    __syncthreads();
    const int groups = (nj + 64 * Q - 1) / (64 * Q);
    const int turns = groups > W ? groups : W, step = turns / W;   // no two wavefronts on one group at a time
    for (int it = 0; it < turns; ++it) {   // same trip count in every lane
        int g = it + wave * step;
        if (g >= turns) g -= turns;
        if (g < groups && iw < ni) {
            const int jg = g * 64 * Q;
            T xj[Q], yj[Q], gx[Q], gy[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int k = jg + q * 64 + lane;
                const T2 v = a.pos[j0 + (k < nj ? k : 0)];
                xj[q] = v.x;
                yj[q] = v.y;
                gx[q] = gy[q] = (T)0;
            }
            const int same = (jg - iw) / 64;   // multiples of 64 both
            const bool pad = jg + 64 * Q > nj || iw + 64 * P > ni;
            if (self) {
                if (pad)
                    pf_sym_group<T, P, Q, true, true>(c, xi, yi, fx, fy, xj, yj, gx, gy, same, ni - iw, nj - jg);
                else
                    pf_sym_group<T, P, Q, true, false>(c, xi, yi, fx, fy, xj, yj, gx, gy, same, 0, 0);
            } else if (pad) {
                pf_sym_group<T, P, Q, false, true>(c, xi, yi, fx, fy, xj, yj, gx, gy, 0, ni - iw, nj - jg);
            } else {
                pf_sym_group<T, P, Q, false, false>(c, xi, yi, fx, fy, xj, yj, gx, gy, 0, 0, 0);
            }
            if (!self) {
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int k = jg + q * 64 + lane;
                    if (k < nj) {
                        T2 v = jsum[k];
                        v.x += gx[q];
                        v.y += gy[q];
                        jsum[k] = v;
                    }
                }
            }
        }
        __syncthreads();   // the sums of this turn's groups are in place
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int k = iw + p * 64 + lane;
        if (k < ni) {
            T2 v;
            v.x = fx[p];
            v.y = fy[p];
            a.part[(size_t)cb * n + i0 + k] = v;
        }
    }
    if (!self)
        for (int k = threadIdx.x; k < nj; k += 64 * W) a.part[(size_t)ca * n + j0 + k] = jsum[k];
}

// F of sorted particle k: its sums over the chunks of each species, weighted, in FP64 and chunk order.
template <typename T>
__global__ void k_pf_sym_reduce(int n, int C, PfLaw law, PfSym<T> a, double *__restrict__ f) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    int s = -1, base = 0;   // the species at place k
    for (int b = 0; b < law.S; ++b) {
        if (k >= base && k < base + a.total[b]) s = b;
        base += a.total[b];
    }
    if (s < 0) return;   // past the last particle
    double fx = 0.0, fy = 0.0;
    int c = 0;
    for (int b = 0; b < law.S; ++b) {
        const int end = c + (a.total[b] + C - 1) / C;
        double sx = 0.0, sy = 0.0;
#pragma unroll 16
        for (; c < end; ++c) {
            const auto v = a.part[(size_t)c * n + k];
            sx += (double)v.x;
            sy += (double)v.y;
        }
        const double w = law.K[s * law.S + b];
        fx += w * sx;
        fy += w * sy;
    }
    const size_t o = 2 * (size_t)a.sid[k];
    f[o] = fx;
    f[o + 1] = fy;
}

// ---------------------------------------------------------------- cells
// Cells of side h, a hair over the cutoff, on a torus of kGrid x kGrid: cell (floor(x / h) mod kGrid, ...), so no
// bounding box is needed; particles a multiple of kGrid cells apart share cells and fail the distance test.  Two
// particles whose working-precision separation passes the cutoff test lie in neighbouring cells: the hair is wider
// than the rounding of that test and of x / h up to kMaxCell cells from the origin.  Inside a cell the particles are
// in ascending order of their index, so the sums do not depend on scheduling.
constexpr int kGrid = 128;
constexpr int kCells = kGrid * kGrid;   // 64 KiB of counters in LDS
constexpr double kMaxCell = 1048576.0;
constexpr int kBinBlock = 1024;

template <typename T>
struct PfCells {
    using T2 = typename Vec2<T>::type;
    int *crowded;           // set: the tiles run instead
    int *start;             // [kCells + 1]
    int *ids;               // [n] particles by cell, in any order
    int *sid, *sp;          // [n] particle and species by cell, ascending
    unsigned short *cell;   // [n] cell of each particle
    T2 *pos;                // [n] as sid
    double inv_h;
};

template <typename T>
__device__ __forceinline__ int pf_cell(T x, T y, double inv_h, bool &ok) {
    const double sx = (double)x * inv_h, sy = (double)y * inv_h;
    ok = fabs(sx) < kMaxCell && fabs(sy) < kMaxCell;   // neither for what is not a number
    return ok ? ((int)floor(sy) & (kGrid - 1)) * kGrid + ((int)floor(sx) & (kGrid - 1)) : 0;
}

// Counting sort by cell in one workgroup: at these sizes a launch costs more than the spread over more compute units
// would save.  kBinAhead particles of a thread are in flight.
constexpr int kBinAhead = 8;

// Too crowded for the cells: nine cells around each particle hold about 9 sum(count^2) pairs in all; above n^2 / 4.7
// (FP64) or n^2 / 6.2 (FP32) of them the tiles are faster.  Evenly filled boxes of r cutoffs a side, tiles and cells,
// us: screened FP64 9,000 particles 107 / 102 at r = 6, 97 / 83 at 7, 20,011 362 / 341 at 5.3, 332 / 259 at 6; inverse
// square FP32 9,000 64 / 68 at 7, 64 / 60 at 8, 20,011 173 / 173 at 6, 173 / 136 at 7.  The line is that of the smaller
// calls; at 100,000 the two meet at r = 4 (screened FP64 10.3 / 10.1 ms, 7.0 / 5.2 at 6) and at 5 (inverse square FP32
// 3.3 / 4.0 at 4.6, 3.3 / 3.0 at 5.3).
template <typename T>
__device__ __forceinline__ bool pf_crowded(unsigned long long squares, unsigned long long n) {
    return (sizeof(T) == 4 ? 56 : 42) * squares > n * n;
}

template <typename T>
__global__ __launch_bounds__(kBinBlock) void k_pf_bin(int n, const double *__restrict__ xy, PfCells<T> a) {
    __shared__ int cnt[kCells];
    __shared__ int wsum[kBinBlock / 64], bad;
    __shared__ unsigned long long crowd;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int c = tid; c < kCells; c += kBinBlock) cnt[c] = 0;
    if (tid == 0) {
        bad = 0;
        crowd = 0;
    }
    __syncthreads();
    {   // a particle per thread shows a crowd before all are counted (m samples: m^2 sum p^2 + m squares)
        const int i = (int)((long long)n * tid / kBinBlock);
        bool ok;
        const int c = pf_cell((T)xy[2 * (size_t)i], (T)xy[2 * (size_t)i + 1], a.inv_h, ok);
        if (!ok) bad = 1;
        const int before = atomicAdd(&cnt[c], 1);   // sum over the samples of 2 before + 1 = sum of the squares
        unsigned sq = 2u * (unsigned)before;
        for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off);
        if (lane == 0) atomicAdd(&crowd, (unsigned long long)sq);
        __syncthreads();
        const bool stop = bad || pf_crowded<T>(crowd, kBinBlock);
        if (stop && tid == 0) *a.crowded = 1;
        if (stop) return;   // uniform in the workgroup
        __syncthreads();
        cnt[c] = 0;
        if (tid == 0) crowd = 0;
        __syncthreads();
    }
    for (int i0 = tid; i0 < n; i0 += kBinBlock * kBinAhead) {
        T x[kBinAhead], y[kBinAhead];
#pragma unroll
        for (int u = 0; u < kBinAhead; ++u) {
            const int i = min(i0 + u * kBinBlock, n - 1);
            x[u] = (T)xy[2 * (size_t)i];
            y[u] = (T)xy[2 * (size_t)i + 1];
        }
#pragma unroll
        for (int u = 0; u < kBinAhead; ++u) {
            const int i = i0 + u * kBinBlock;
            if (i >= n) continue;
            bool ok;
            const int c = pf_cell(x[u], y[u], a.inv_h, ok);
            if (!ok) bad = 1;
            a.cell[i] = (unsigned short)c;
            atomicAdd(&cnt[c], 1);
        }
    }
    __syncthreads();
    constexpr int kOwn = kCells / kBinBlock;   // consecutive cells of a thread
    int own[kOwn], sum = 0;
    unsigned long long sq = 0;
#pragma unroll
    for (int u = 0; u < kOwn; ++u) {
        own[u] = cnt[tid * kOwn + u];
        sum += own[u];
        sq += (unsigned long long)own[u] * own[u];
    }
    int incl = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    if (lane == 63) wsum[wave] = incl;
    if (sq) atomicAdd(&crowd, sq);
    __syncthreads();
    int at = incl - sum;
    for (int w = 0; w < wave; ++w) at += wsum[w];
#pragma unroll
    for (int u = 0; u < kOwn; ++u) {
        a.start[tid * kOwn + u] = at;
        cnt[tid * kOwn + u] = at;
        at += own[u];
    }
    if (tid == kBinBlock - 1) a.start[kCells] = n;
    const bool crowded = bad || pf_crowded<T>(crowd, (unsigned long long)n);
    if (tid == 0) *a.crowded = crowded ? 1 : 0;
    if (crowded) return;   // uniform in the workgroup
    __syncthreads();
    for (int i0 = tid; i0 < n; i0 += kBinBlock * kBinAhead) {
        int c[kBinAhead];
#pragma unroll
        for (int u = 0; u < kBinAhead; ++u) c[u] = a.cell[min(i0 + u * kBinBlock, n - 1)];
#pragma unroll
        for (int u = 0; u < kBinAhead; ++u)
            if (i0 + u * kBinBlock < n) a.ids[atomicAdd(&cnt[c[u]], 1)] = i0 + u * kBinBlock;
    }
}

// Each particle to its place: its cell's start and the number of smaller indices in the cell.
template <typename T>
__global__ __launch_bounds__(kPfBlock) void k_pf_place(int n, const double *__restrict__ xy,
                                                       const int32_t *__restrict__ species, PfCells<T> a) {
    const int e = blockIdx.x * kPfBlock + threadIdx.x;
    if (e >= n || *a.crowded) return;
    const int i = a.ids[e], c = a.cell[i];
    const int b = a.start[c], end = a.start[c + 1];
    int at = b;
#pragma unroll 8
    for (int k = b; k < end; ++k) at += a.ids[k] < i ? 1 : 0;
    typename Vec2<T>::type v;
    v.x = (T)xy[2 * (size_t)i];
    v.y = (T)xy[2 * (size_t)i + 1];
    a.pos[at] = v;
    a.sid[at] = i;
    a.sp[at] = species[i];
}

// LANES lanes per particle, each every LANES-th one of its 3 x 3 cells (three runs of consecutive particles, or up to
// six where the torus closes).  A third of them is in range and a law costs many times the test, so hits are noted and
// evaluated together as in the tiles; a lane's sum keeps their order, the lanes are added in FP64.
// Waits for its chains of loads, so small calls take more lanes: 20,011 particles, screened law, FP64, whole call 61 us
// with 4 lanes, 50 with 8, 47 with 16, 51 with 32 (140 us by tiles); 65,536 109, 104, 110 and 126 (970 by tiles).
constexpr int kCellsWide = 32768;   // 16 lanes up to here, 8 above

template <typename T, int LAW, int LANES>
__global__ __launch_bounds__(kPfBlock) void k_pf_cells(int n, PfCells<T> a, PfLaw law, double *__restrict__ f) {
    __shared__ T kw[BD_MAX_SPECIES * BD_MAX_SPECIES];
    __shared__ int hit[kPfHits][kPfBlock];
    if (*a.crowded) return;
    const int S = law.S, tid = threadIdx.x;
    for (int k = tid; k < S * S; k += kPfBlock) kw[k] = (T)law.K[k];
    __syncthreads();
    const PfConst<T> c(law);
    const int g = blockIdx.x * (kPfBlock / LANES) + tid / LANES, lane = tid & (LANES - 1);
    const int i = min(g, n - 1);
    const auto pi = a.pos[i];
    const int si = a.sp[i] * S;
    bool ok;
    const int ci = pf_cell(pi.x, pi.y, a.inv_h, ok), cx = ci & (kGrid - 1), cy = ci / kGrid;
    T ax = (T)0, ay = (T)0;
    int cnt = 0;
    auto evaluate = [&]() {
        for (int h = 0; __ballot(h < cnt) != 0; ++h) {
            if (h < cnt) {
                const int k = hit[h][tid];
                const auto q = a.pos[k];
                const T dx = pi.x - q.x, dy = pi.y - q.y;
                const int sj = a.sp[k];   // out of range: not counted, as in the tiles
                const T w = (unsigned)sj < (unsigned)S ? kw[si + sj] * law_factor<LAW>(dx * dx + dy * dy, c) : (T)0;
                ax += dx * w;
                ay += dy * w;
            }
        }
        cnt = 0;
    };
    auto run = [&](int k, int end) {   // every lane is here; a run may be empty
        constexpr int kU = 4;
        for (; __ballot(k < end) != 0; k += kU * LANES) {
            typename Vec2<T>::type q[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) q[u] = a.pos[k + u * LANES < end ? k + u * LANES : i];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int ku = k + u * LANES;
                const T dx = pi.x - q[u].x, dy = pi.y - q[u].y;
                const bool in = ku < end && ku != i && !(dx * dx + dy * dy > c.cut2);
                if (in) hit[cnt++][tid] = ku;
                if (__ballot(cnt == kPfHits) != 0) evaluate();
            }
        }
    };
    const bool split = cx == 0 || cx == kGrid - 1;
    for (int r = -1; r <= 1; ++r) {
        const int *row = a.start + ((cy + r) & (kGrid - 1)) * kGrid;
        const int x0 = cx == 0 ? 0 : cx - 1, x1 = cx == kGrid - 1 ? cx : cx + 1;
        run(row[x0] + lane, row[x1 + 1]);
        if (__ballot(split) != 0) {   // the cell on the other side
            const int x = cx == 0 ? kGrid - 1 : 0;
            run(row[x] + lane, split ? row[x + 1] : 0);
        }
    }
    evaluate();
    double fx = (double)ax, fy = (double)ay;
    for (int off = 1; off < LANES; off <<= 1) {
        fx += __shfl_xor(fx, off);
        fy += __shfl_xor(fy, off);
    }
    if (lane == 0 && g < n) {
        const size_t o = 2 * (size_t)a.sid[i];
        f[o] = fx;
        f[o + 1] = fy;
    }
}

size_t pf_value_bytes(int precision) { return precision == BD_PREC_FP32 ? sizeof(float2) : sizeof(double2); }

int pf_check(int32_t n, const double *xy, const int32_t *species, const bd_force_params *fp, int32_t precision,
             const double *f_out, PfLaw &law) {
    if (n < 1 || !xy || !species || !fp || !f_out || !fp->K) return BD_ERR_INVALID_ARG;
    if (precision != BD_PREC_FP32 && precision != BD_PREC_FP64) return BD_ERR_INVALID_ARG;
    if (fp->S < 1 || fp->S > BD_MAX_SPECIES) return BD_ERR_INVALID_ARG;
    if (fp->kind != BD_FORCE_POWER && fp->kind != BD_FORCE_SCREENED) return BD_ERR_INVALID_ARG;
    if (fp->kind == BD_FORCE_POWER && !(std::isfinite(fp->q) && fp->q > 0.0)) return BD_ERR_INVALID_ARG;
    if (fp->kind == BD_FORCE_SCREENED && !(std::isfinite(fp->A) && std::isfinite(fp->lambda) && fp->lambda > 0.0))
        return BD_ERR_INVALID_ARG;
    if (!std::isfinite(fp->cutoff)) return BD_ERR_INVALID_ARG;
    std::memset(&law, 0, sizeof(law));
    law.kind = fp->kind;
    law.S = fp->S;
    law.q = fp->q;
    law.A = fp->A;
    law.lam = fp->kind == BD_FORCE_SCREENED ? fp->lambda : 1.0;
    law.cutoff = fp->cutoff;
    for (int k = 0; k < fp->S * fp->S; ++k) {
        if (!std::isfinite(fp->K[k])) return BD_ERR_INVALID_ARG;
        law.K[k] = fp->K[k];
    }
    return BD_OK;
}

// How a call runs; depends on n, the precision and the law only.
struct PfPlan {
    bool rows;    // rows layout
    int sym;      // chunk length of the sym layout (0: another layout)
    bool cells;   // cells, with the tiles behind them
    int J;        // tiles layout: j splits
    size_t bytes;
};

constexpr int kSymMin = 16384;

constexpr size_t pf_align(size_t b) { return (b + 255) / 256 * 256; }

// Places of the cells' arrays in the working memory, the flag first (the tiles' sums, if it comes to them, take what
// follows it); returns the bytes.
template <typename T>
size_t pf_cells_at(int n, const PfLaw &law, unsigned char *base, PfCells<T> &a) {
    size_t o = 256;
    auto take = [&](auto *&p, size_t count) {
        p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(base + o);
        o += pf_align(count * sizeof(*p));
    };
    a.crowded = reinterpret_cast<int *>(base);
    take(a.start, kCells + 1);
    take(a.ids, n);
    take(a.sid, n);
    take(a.sp, n);
    take(a.cell, n);
    take(a.pos, n);
    a.inv_h = 1.0 / (law.cutoff * (sizeof(T) == 4 ? 1.0 + 1e-5 : 1.0 + 1e-9));
    return o;
}

constexpr size_t kPfPartBytes = size_t(32) << 20;   // most working memory of a call that more than one split needs

// Most particles of the cells layout: its sort is one workgroup's, its arrays stay below kPfPartBytes.
constexpr int kCellsMax = 262144;

// Places of the sym layout's arrays; returns the bytes.
template <typename T>
size_t pf_sym_at(int n, int S, int C, unsigned char *base, PfSym<T> &a) {
    size_t o = 0;
    auto take = [&](auto *&p, size_t count) {
        p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(base + o);
        o += pf_align(count * sizeof(*p));
    };
    take(a.count, (size_t)((n + kSortBlock - 1) / kSortBlock) * BD_MAX_SPECIES);
    take(a.total, BD_MAX_SPECIES);
    take(a.sid, n);
    take(a.pos, n);
    take(a.part, (size_t)(n / C + S) * n);
    return o;
}

// Particles i per lane of the tiles: one LDS read of a j serves them all.  Four for the shortest pair loop
// (FP32 inverse square: 9 instructions); two where a pair is longer or notes its hits.
template <typename T, int LAW, bool CUT>
constexpr int pf_per_lane() { return sizeof(T) == 4 && LAW == PF_Q2 && !CUT ? 4 : 2; }

PfPlan pf_plan(int n, int precision, const PfLaw &law) {
    PfPlan p{};
    const bool cut = law.cutoff > 0.0;
    // Rows up to these sizes.  Measured, rows against tiles, two species, us: no cutoff, inverse square, FP64
    // 27 / 33 at 5,000, 36 / 47 at 6,000, 60 / 49 at 8,192, FP32 25 / 34 at 6,000, 49 / 35 at 8,192; screened FP64
    // 72 / 80 at 5,000, 165 / 137 at 8,192.  With a cutoff, where rows evaluates the law for the lanes out of range
    // too, rows against cells (cutoff 12, 0.45 of the area covered, three species): inverse square FP64 23 / 27 at
    // 4,000, FP32 22 / 29; screened FP64 20 / 30 at 2,000, 55 / 31 at 4,000, FP32 37 / 33 at 4,000; but with cutoffs
    // of a fifth of the box and more, which the cells leave to the tiles, rows 53 / 89 to 139 at 3,700 (screened FP64).
    const bool q2 = law.kind == BD_FORCE_POWER && law.q == 2.0;
    p.rows = n <= (cut ? 4096 : 6144);
    if (p.rows) return p;
    // Every pair once above 16,384 particles, where the chunks' sums fit the working memory: the smallest chunk that
    // lets them (smaller tiles leave fewer compute units waiting at the end).  Tiles against sym, three species, us:
    // FP32 86 / 94 at 16,001, 130 / 98 at 18,000, 118 / 117 at 20,011, 245 / 176 at 30,000 (chunks of 256), 472 / 363
    // at 43,000 (512), 941 / 685 at 62,000 (1024), 957 / 754 at 65,536 (1280; 963 with four particles a lane, which
    // leave a second round of workgroups there).  Chunks of 1280, FP32 only, are the last that fit, with two species
    // for 64,031 to 71,680: 1059 / 802 at 64,100, 1148 / 809 at 67,000, 1276 / 905 at 70,500, 1289 / 910 at 71,600; one
    // species 1188 / 822 at 68,000, eight 1135 / 913 at 66,000.  FP64 149 / 156 at 16,001, 195 / 161 at 18,000, 235 /
    // 205 at 20,011, 506 / 372 at 30,000, 1006 / 701 at 43,000, 1107 / 752 at 44,500, and above, where chunks of 1280
    // fill the device unevenly, 1309 / 1424 at 49,000.
    const bool fp32 = precision == BD_PREC_FP32;
    if (q2 && !cut && n > kSymMin) {
        for (int C : {256, 512, 1024, 1280}) {
            PfSym<float> a32;
            PfSym<double> a64;
            const size_t b = fp32 ? pf_sym_at(n, law.S, C, nullptr, a32) : pf_sym_at(n, law.S, C, nullptr, a64);
            if (b > kPfPartBytes || (!fp32 && C > 1024)) continue;
            p.sym = C;
            p.bytes = b;
            return p;
        }
    }
    p.cells = cut && n <= kCellsMax;
    const bool four = precision == BD_PREC_FP32 && q2 && !cut;
    const long long per_group = (long long)kPfBlock * (four ? 4 : 2), nb = (n + per_group - 1) / per_group;
    // enough splits to fill the device, of at least kPfBlock j, as far as the working memory reaches
    long long J = (kPfTargetGroups + nb - 1) / nb;
    const size_t row = (size_t)n * pf_value_bytes(precision);
    J = std::min({J, (long long)kPfMaxSplits, ((long long)n + kPfBlock - 1) / kPfBlock,
                  (long long)(kPfPartBytes / row)});
    p.J = (int)std::max(1ll, J);
    p.bytes = p.J * row;
    if (p.cells) {
        PfCells<float> a32;
        PfCells<double> a64;
        const size_t c = fp32 ? pf_cells_at(n, law, nullptr, a32) : pf_cells_at(n, law, nullptr, a64);
        const size_t most = kPfPartBytes - 256;
        p.J = std::min(p.J, (int)(most / row));
        p.bytes = std::max(256 + p.J * row, c);
    }
    return p;
}

template <typename T, int LAW, bool CUT>
void pf_launch(int n, const double *xy, const int32_t *species, const PfLaw &law, double *f_out, hipStream_t stream,
               void *part, const PfPlan &p) {
    using T2 = typename Vec2<T>::type;
    const dim3 block(kPfBlock);
    if (p.rows) {
        constexpr int kWaves = kPfBlock / 64;
        hipLaunchKernelGGL((k_pf_rows<T, LAW, CUT>), dim3((n + kWaves - 1) / kWaves), block, 0, stream, n, xy,
                           species, law, f_out);
        return;
    }
    if constexpr (LAW == PF_Q2 && !CUT) {
        if (p.sym) {
            constexpr int Q = sizeof(T) == 4 ? 2 : 1;
            const int C = p.sym, nc = n / C + law.S, nb = (n + kSortBlock - 1) / kSortBlock;
            PfSym<T> a;
            pf_sym_at(n, law.S, C, (unsigned char *)part, a);
            hipLaunchKernelGGL(k_pf_count, dim3(nb), dim3(kSortBlock), 0, stream, n, law.S, species, a.count);
            hipLaunchKernelGGL(k_pf_sort<T>, dim3(nb), dim3(kSortBlock), 0, stream, n, law.S, xy, species, a);
            auto tiles = [&](auto kern, int waves) {
                hipLaunchKernelGGL(kern, dim3(nc * (nc + 1) / 2), dim3(64 * waves), 0, stream, n, law, a);
            };
            if (C == 256)
                tiles(k_pf_sym<T, 4, 1, Q>, 1);
            else if (C == 512)
                tiles(k_pf_sym<T, 4, 2, Q>, 2);
            else if (C == 1024)
                tiles(k_pf_sym<T, 4, 4, Q>, 4);
            else if constexpr (sizeof(T) == 4)   // five per lane: six workgroups on a compute unit
                tiles(k_pf_sym<T, 5, 4, Q>, 4);
            hipLaunchKernelGGL(k_pf_sym_reduce<T>, dim3((n + 255) / 256), dim3(256), 0, stream, n, C, law, a, f_out);
            return;
        }
    }
    constexpr int P = pf_per_lane<T, LAW, CUT>();
    const dim3 grid((n + kPfBlock * P - 1) / (kPfBlock * P), p.J);
    const int *crowded = nullptr;
    if constexpr (CUT) {
        if (p.cells) {
            PfCells<T> a;
            pf_cells_at(n, law, (unsigned char *)part, a);
            hipLaunchKernelGGL(k_pf_bin<T>, dim3(1), dim3(kBinBlock), 0, stream, n, xy, a);
            hipLaunchKernelGGL(k_pf_place<T>, dim3((n + kPfBlock - 1) / kPfBlock), block, 0, stream, n, xy, species, a);
            auto sums = [&](auto kern, int lanes) {
                const int per = kPfBlock / lanes;
                hipLaunchKernelGGL(kern, dim3((n + per - 1) / per), block, 0, stream, n, a, law, f_out);
            };
            n <= kCellsWide ? sums(k_pf_cells<T, LAW, 16>, 16) : sums(k_pf_cells<T, LAW, 8>, 8);
            crowded = a.crowded;
            part = (unsigned char *)part + 256;
        }
    }
    hipLaunchKernelGGL((k_pf_tiles<T, LAW, CUT, P>), grid, block, 0, stream, n, p.J, xy, species, law, (T2 *)part,
                       crowded);
    hipLaunchKernelGGL(k_pf_reduce<T>, dim3((n + 255) / 256), dim3(256), 0, stream, n, p.J, (const T2 *)part, f_out,
                       crowded);
}

template <typename T>
void pf_launch_law(int n, const double *xy, const int32_t *species, const PfLaw &law, double *f_out,
                   hipStream_t stream, void *part, const PfPlan &p) {
    const bool cut = law.cutoff > 0.0;
    auto go = [&](auto form) {
        constexpr int LAW = decltype(form)::value;
        if (cut)
            pf_launch<T, LAW, true>(n, xy, species, law, f_out, stream, part, p);
        else
            pf_launch<T, LAW, false>(n, xy, species, law, f_out, stream, part, p);
    };
    if (law.kind == BD_FORCE_SCREENED)
        go(std::integral_constant<int, PF_SCREENED>{});
    else if (law.q == 2.0)
        go(std::integral_constant<int, PF_Q2>{});
    else
        go(std::integral_constant<int, PF_POWER>{});
}

// Enqueues the call's kernels on `stream` with `part` as the split sums.
int pf_enqueue(int32_t n, const double *xy, const int32_t *species, const PfLaw &law, int32_t precision,
               double *f_out, hipStream_t stream, void *part, const PfPlan &p) {
    if (precision == BD_PREC_FP32)
        pf_launch_law<float>(n, xy, species, law, f_out, stream, part, p);
    else
        pf_launch_law<double>(n, xy, species, law, f_out, stream, part, p);
    return hipGetLastError() == hipSuccess ? BD_OK : BD_ERR_DEVICE;
}

}  // namespace

extern "C" int bd_pair_forces_dev(int32_t n, const double *xy, const int32_t *species, const bd_force_params *fp,
                                  int32_t precision, double *f_out, void *stream) {
    PfLaw law;
    const int rc = pf_check(n, xy, species, fp, precision, f_out, law);
    if (rc != BD_OK) return rc;
    const hipStream_t st = (hipStream_t)stream;
    const PfPlan p = pf_plan(n, precision, law);
    void *part = nullptr;
    if (p.bytes && hipMalloc(&part, p.bytes) != hipSuccess) {
        (void)hipGetLastError();
        return BD_ERR_OOM;
    }
    int out = pf_enqueue(n, xy, species, law, precision, f_out, st, part, p);
    if (hipStreamSynchronize(st) != hipSuccess) out = BD_ERR_DEVICE;
    if (part && hipFree(part) != hipSuccess) out = BD_ERR_DEVICE;
    return out;
}

// ------------------------------------------------------------------ no-allocation variant
// For callers that cannot allocate device memory (code under HIP graph capture,
// serving loops, harnesses that forbid hipMalloc): the split sums live in a
// fixed device array of kScratchBytes, one copy per GPU, held until the
// process ends.  Its device address is looked up once per device (with that
// device current) on the first call there; kernels receive that address,
// never the array's host-side name.
namespace {

constexpr size_t kScratchBytes = kPfPartBytes;
constexpr int kMaxDevices = 64;

__device__ __align__(256) unsigned char scratch[kScratchBytes];

std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices];

// Device address of this device's scratch array, or nullptr on failure.
void *scratch_for_current_device() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return nullptr;
    }
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}

}  // namespace

extern "C" int bd_pair_forces_dev_noalloc(int32_t n, const double *xy, const int32_t *species,
                                          const bd_force_params *fp, int32_t precision, double *f_out, void *stream) {
    PfLaw law;
    const int rc = pf_check(n, xy, species, fp, precision, f_out, law);
    if (rc != BD_OK) return rc;
    const PfPlan p = pf_plan(n, precision, law);
    if (p.bytes > kScratchBytes) {
        std::fprintf(stderr, "bd_pair_forces_dev_noalloc: n = %d needs %zu bytes of scratch, more than its %zu\n",
                     (int)n, p.bytes, kScratchBytes);
        return BD_ERR_INVALID_ARG;
    }
    void *part = scratch_for_current_device();
    if (!part) return BD_ERR_DEVICE;
    // every split sum that the reduction reads is written first: nothing to clear
    return pf_enqueue(n, xy, species, law, precision, f_out, (hipStream_t)stream, part, p);
}
