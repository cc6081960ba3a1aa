// S1: cell list and neighbour lists (the chaining mesh of Sec. 3.3 with one
// interaction list per step that every later pass reuses).
//
// 1. validate + reduce H (deterministic two-level reduction)
// 2. key = Morton code of the particle's cell; stable radix sort -> perm
// 3. gather sorted x, y, z, H into one double4 per particle; cell ranges
// 4. walk: a wavefront takes a few consecutive particles, visits the cells of
//    the hierarchy level matched to their supports and finds the j with r^2 < H_i^2 (the
//    gather set, self excluded), and among them the j with r^2 >= H_j^2: j
//    reaches i only through i's larger support, so the pair is an "extra"
//    of j. Hits go to a capped scratch row, with exact counts.
// 5. exclusive scans of both counts give every particle its output slots;
//    the scratch rows are compacted, and rows past the cap walked again
// 6. the extras, grouped by i, are transposed into rows per j, each row
//    ascending in i (placed by rank, so the atomic slot counters of the
//    scatter decide nothing). The lists, and every sum over them, are the
//    same bit for bit from run to run.
#include <math.h>

#include <algorithm>

#include "crk_internal.h"

namespace crk {
namespace {

__global__ __launch_bounds__(kBlock) void k_validate(const double *x, const double *y,
                                                     const double *z, const double *H, int64_t n,
                                                     double L, double *part /* [nblk][3] */,
                                                     int *flags /* [nblk]: bits as in k_validate_final */) {
    __shared__ int sflags;
    __shared__ double smax[kBlock], smin[kBlock], ssum[kBlock];
    double hmax = 0.0, hmin = INFINITY, hsum = 0.0;
    int nf = 0, rg = 0, bh = 0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock) {
        double a = x[i], b = y[i], c = z[i], h = H[i];
        if (!isfinite(a) || !isfinite(b) || !isfinite(c) || !isfinite(h)) {
            nf = 1;
            continue;
        }
        if (a < 0.0 || a >= L || b < 0.0 || b >= L || c < 0.0 || c >= L) rg = 1;
        if (!(h > 0.0)) bh = 1;
        hmax = fmax(hmax, h);
        hmin = fmin(hmin, h);
        hsum += h;
    }
    smax[threadIdx.x] = hmax;
    smin[threadIdx.x] = hmin;
    ssum[threadIdx.x] = hsum;
    if (threadIdx.x == 0) sflags = 0;
    __syncthreads();
    if (nf | rg | bh) atomicOr(&sflags, nf | rg << 1 | bh << 2);
    for (int s = kBlock / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + s]);
            smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + s]);
            ssum[threadIdx.x] += ssum[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[blockIdx.x * 3 + 0] = smax[0];
        part[blockIdx.x * 3 + 1] = smin[0];
        part[blockIdx.x * 3 + 2] = ssum[0];
        flags[blockIdx.x] = sflags;
    }
}

// what k_validate_final finds: extrema and sum of H, and the flags
// (bit 0 non-finite input, bit 1 position outside [0, L), bit 2 H <= 0)
struct Checks {
    double hmax, hmin, hsum;
    int flags;
};

// Final reduction of the (at most 1024) block partials by one block, in a
// fixed tree order: to host (pinned memory, read once the stream is done), or
// as the status of a graph-mode step in st (its bits as in Checks, bit 3
// H >= L/2). boff: the offsets 0, n of a single box.
__global__ __launch_bounds__(1024) void k_validate_final(const double *part, const int *flags, int nblk, double L,
                                                         int64_t *boff, int64_t n, Checks *host, GraphStat *st) {
    __shared__ double smax[1024], smin[1024], ssum[1024];
    __shared__ int sflags;
    const int t = threadIdx.x;
    smax[t] = t < nblk ? part[t * 3 + 0] : 0.0;
    smin[t] = t < nblk ? part[t * 3 + 1] : INFINITY;
    ssum[t] = t < nblk ? part[t * 3 + 2] : 0.0;
    if (t == 0) sflags = 0;
    __syncthreads();
    if (t < nblk && flags[t]) atomicOr(&sflags, flags[t]);
    for (int s = 512; s > 0; s >>= 1) {
        if (t < s) {
            smax[t] = fmax(smax[t], smax[t + s]);
            smin[t] = fmin(smin[t], smin[t + s]);
            ssum[t] += ssum[t + s];
        }
        __syncthreads();
    }
    if (t != 0) return;
    if (boff) {
        boff[0] = 0;
        boff[1] = n;
    }
    if (host) *host = Checks{smax[0], smin[0], ssum[0], sflags};
    if (st) {
        int e = sflags | (!(smin[0] > 0.0) ? 4 : 0);
        if (!(sflags & 1) && !(smax[0] < 0.5 * L)) e |= 8;
        st->input_error = e;
        st->overflow = 0;
        st->clear = 0;
    }
}

// Graph mode cannot stop on invalid input before the walk, so such a
// particle is moved to a fixed in-box point (the R3 low-discrepancy sequence
// of its index) with a vanishing support: every later access stays in
// bounds, and the step's status reports the error.
__device__ __forceinline__ bool invalid_particle(double x, double y, double z, double h, double L) {
    return !(x >= 0.0 && x < L && y >= 0.0 && y < L && z >= 0.0 && z < L && h > 0.0 && h < 0.5 * L);
}

__device__ __forceinline__ double4 stand_in(int64_t i, double L) {
    double t = (double)i;
    return make_double4(L * (t * 0.8191725133961645 - floor(t * 0.8191725133961645)),
                        L * (t * 0.6710436067037893 - floor(t * 0.6710436067037893)),
                        L * (t * 0.5497004779019703 - floor(t * 0.5497004779019703)), 1e-9 * L);
}

__device__ __forceinline__ int cell_of(double x, double inv_c, int nc) {
    int k = (int)floor(x * inv_c);
    return k < 0 ? 0 : (k >= nc ? nc - 1 : k);
}

// key = (box << 3 bits) | Morton code of the particle's finest cell; the box
// is found by bisection of the batch's particle offsets. per_block particles a
// block (a multiple of its threads); counts: the first digits of the block's
// keys counted for the sort (null: not wanted)
__global__ __launch_bounds__(kBlock) void k_keys(const double *x, const double *y, const double *z,
                                                 int64_t n, double inv_c, int nc, int bits,
                                                 const int64_t *__restrict__ boff, int nboxes,
                                                 const double *H, double L, uint32_t *key, int32_t *val,
                                                 int64_t per_block, int32_t *counts) {
    __shared__ int cnt[256];
    static_assert(kBlock == 256, "a thread per digit");
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * per_block + threadIdx.x;
    for (int64_t i = i0; i < i0 + per_block && i < n; i += kBlock) {
        int lo = 0, hi = nboxes - 1;
        while (lo < hi) {
            int mid = (lo + hi + 1) >> 1;
            if (boff[mid] <= i) lo = mid;
            else hi = mid - 1;
        }
        double px = x[i], py = y[i], pz = z[i];
        if (H && invalid_particle(px, py, pz, H[i], L)) {
            double4 s = stand_in(i, L);
            px = s.x;
            py = s.y;
            pz = s.z;
        }
        uint32_t m = morton3(cell_of(px, inv_c, nc), cell_of(py, inv_c, nc), cell_of(pz, inv_c, nc));
        m |= (uint32_t)lo << (3 * bits);
        key[i] = m;
        val[i] = (int32_t)i;
        if (counts) atomicAdd(&cnt[m & 255u], 1);
    }
    if (!counts) return;
    __syncthreads();
    counts[(int64_t)blockIdx.x * 256 + threadIdx.x] = cnt[threadIdx.x];
}

// sorted particles, the permutation for the caller, the walk's counts cleared
// (the extras' and that of the long rows), and the ntot entries of both cell
// tables cleared (16-byte aligned, four entries a thread; the launch covers
// both)
__global__ __launch_bounds__(kBlock) void k_gather_sorted(const double *x, const double *y,
                                                          const double *z, const double *H,
                                                          const int32_t *perm, int64_t n,
                                                          int stand_ins, double L, double4 *posH,
                                                          int32_t *perm_out, int32_t *cbeg, int32_t *cend,
                                                          int64_t ntot, int32_t *ecnt, int32_t *longs) {
    int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k == 0) longs[0] = 0;
    const int4 zero = make_int4(0, 0, 0, 0);
    if (4 * k + 4 <= ntot) {
        ((int4 *)cbeg)[k] = zero;
        ((int4 *)cend)[k] = zero;
    } else {
        for (int64_t e = 4 * k; e < ntot; e++) cbeg[e] = cend[e] = 0;
    }
    if (k >= n) return;
    int32_t i = perm[k];
    perm_out[k] = i;
    ecnt[k] = 0;
    double4 p = make_double4(x[i], y[i], z[i], H[i]);
    if (stand_ins && invalid_particle(p.x, p.y, p.z, p.w, L)) p = stand_in(i, L);
    posH[k] = p;
}

// graph mode: lists longer than the recorded capacity (tot: their lengths)
// empty every row (so that the fills below stay in bounds) and raise the
// overflow flag
__global__ __launch_bounds__(kBlock) void k_graph_cap(const int64_t *tot, int64_t gcap, int64_t ecap, GraphStat *st,
                                                      int64_t n, int64_t *goff, int64_t *eoff, int32_t *ng) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x, G = tot[0], E = tot[1];
    const int o = (G > gcap || E > ecap) ? 1 : 0;
    if (i == 0) {
        st->overflow = o;
        st->clear = o;
        st->n_gather = o ? 0 : G;
        st->n_extra = o ? 0 : E;
    }
    if (i > n || !o) return;
    goff[i] = 0;
    eoff[i] = 0;
    if (i < n) ng[i] = 0;
}

// the extras' counts and the number of long rows before a walk (16-byte
// aligned, four entries a thread)
__global__ __launch_bounds__(kBlock) void k_zero_counts(int32_t *ecnt, int64_t n, int32_t *longs) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t == 0) longs[0] = 0;
    if (4 * t + 4 <= n) ((int4 *)ecnt)[t] = make_int4(0, 0, 0, 0);
    else
        for (int64_t e = 4 * t; e < n; e++) ecnt[e] = 0;
}

// sorted-index range of every cell of every level (a level-k cell is the set
// of particles whose fine Morton code shifted right by 3k is its id)
__global__ __launch_bounds__(kBlock) void k_tables(const uint32_t *skey, int64_t n, Levels v,
                                                   int32_t *cbeg, int32_t *cend) {
    int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= n) return;
    uint32_t key = skey[k];
    uint32_t prev = k > 0 ? skey[k - 1] : 0u, next = k + 1 < n ? skey[k + 1] : 0u;
    const int64_t base = box_base(v, k);
    const uint32_t mort = key & (uint32_t)(((uint64_t)1 << (3 * v.bits)) - 1);
    for (int l = 0; l <= v.bits; l++) {
        // a cell of level l is identified by key >> 3l (box bits included)
        uint32_t id = key >> (3 * l);
        uint32_t loc = mort >> (3 * l);
        if (k == 0 || (prev >> (3 * l)) != id) cbeg[base + v.off[l] + loc] = (int32_t)k;
        if (k == n - 1 || (next >> (3 * l)) != id) cend[base + v.off[l] + loc] = (int32_t)(k + 1);
    }
}

// The walk of one particle by a group of G lanes (the rows over the scratch
// rows' slots; the first walk below shares a wavefront among several
// particles). CULL: the walked range lies within half a period of i, so every
// particle of an (unwrapped) cell has its nearest image in that cell's image:
// the separation is (x_i - x_j) + c with c in {-L, 0, L} fixed per cell, the
// same two roundings the minimum-image rule makes, and cells wholly outside
// the (slightly widened) support are skipped. Otherwise each separation takes
// the minimum-image rule.
//
// The group lists its non-empty, non-skipped cells as ranges of sorted
// particles (in walk order: cells z-major, then y, then x; up to
// walk_ranges<G>() at a time, in LDS, each with the code of its periodic image
// shift) and then takes the concatenated candidates G at a time across cell
// boundaries; a ballot over the group orders the hits as a serial walk would.
//
// The group first fills its axis tables (fill_axes); a listed cell then
// costs three table reads, and its range carries the one-byte code of its
// image shift (the 27 shift triples are a table of the block).

// cell ranges a group lists at a time: four steps of G cells, at most 64
template <int G>
__host__ __device__ constexpr int walk_ranges() {
    return 4 * G > 64 ? 64 : 4 * G;
}

// the 27 image shift triples (dx, dy, dz) by code cx + 3 cy + 9 cz
__device__ __forceinline__ void fill_shifts(double (*sh)[3], double L) {
    const int c = threadIdx.x;
    if (c < 27) {
        const int q[3] = {c % 3, (c / 3) % 3, c / 9};
#pragma unroll
        for (int a = 0; a < 3; a++) sh[c][a] = q[a] == 1 ? L : (q[a] == 2 ? -L : 0.0);
    }
}

template <int G, bool CULL>
__device__ __forceinline__ void walk_row_flat(const double4 *__restrict__ posH, int64_t i,
                                              const double4 &pi, int l, int gshift, uint32_t below,
                                              const Levels &v, const int32_t *__restrict__ cb,
                                              const int32_t *__restrict__ ce_, int nck, int lx, int ly,
                                              int lz, int mx, int my, int mz, double cs, double Hc2,
                                              int64_t first, int32_t *gidx, int32_t *efill, int32_t *etmp,
                                              int32_t *sb, int32_t *sc, uint8_t *scode, AxisTab &tab,
                                              const double (*shifts)[3]) {
    int32_t cg = 0;
    constexpr int NR = walk_ranges<G>();
    const double H2 = pi.w * pi.w;
    const int ncell = mx * my * mz;
    // 1. axis tables
    fill_axes<G, CULL, false>(tab, pi, l, lx, ly, lz, mx, my, mz, nck, cs, v.L);
    const uint32_t dx_ = div16(mx), dy_ = div16(my);
    int c0 = 0;
    while (c0 < ncell) {
        // 2. list up to NR non-empty cells, G cells per step
        int nr = 0, cum = 0;
        while (c0 < ncell && nr + G <= NR) {
            const int cidx = c0 + l;
            int jb = 0, len = 0, code = 0;
            if (cidx < ncell) {
                const int t = (int)(((uint32_t)cidx * dx_) >> 16);
                const int e = cidx - t * mx;
                const int a = (int)(((uint32_t)t * dy_) >> 16);
                const int b = t - a * my;
                bool keep = true;
                if (CULL) keep = (tab.g2[2][a] + tab.g2[1][b]) + tab.g2[0][e] <= Hc2;
                if (keep) {
                    const uint32_t ix = tab.id[0][e], iy = tab.id[1][b], iz = tab.id[2][a];
                    const uint32_t id = (ix | iy | iz) & 0x3fffffffu;
                    code = (int)(ix >> 30) + 3 * (int)(iy >> 30) + 9 * (int)(iz >> 30);
                    jb = cb[id];
                    len = ce_[id] - jb;
                }
            }
            int tot;
            const int pre = group_excl_scan<G>(len, l, tot);
            const bool has = len > 0;
            const uint32_t hm = (uint32_t)((__ballot(has) >> gshift) & (((uint64_t)1 << G) - 1));
            if (has) {
                const int pos = nr + __popc(hm & below);
                sb[pos] = jb;
                sc[pos] = cum + pre;
                scode[pos] = (uint8_t)code;
            }
            nr += __popc(hm);
            cum += tot;
            c0 += G;
        }
        if (l == 0) sc[nr] = cum;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // 3. the listed candidates, G at a time
        int r = 0;
        for (int f0 = 0; f0 < cum; f0 += G) {
            const int f = f0 + l;
            bool hit = false, extra = false;
            int j = 0;
            if (f < cum) {
                while (sc[r + 1] <= f) r++;
                j = sb[r] + (f - sc[r]);
                const double4 pj = posH[j];
                double dx, dy, dz;
                if (CULL) {
                    const double *sh = shifts[scode[r]];
                    dx = (pi.x - pj.x) + sh[0];
                    dy = (pi.y - pj.y) + sh[1];
                    dz = (pi.z - pj.z) + sh[2];
                } else {
                    dx = min_image(pi.x - pj.x, v.L, v.hL);
                    dy = min_image(pi.y - pj.y, v.L, v.hL);
                    dz = min_image(pi.z - pj.z, v.L, v.hL);
                }
                const double r2 = r2_exact(dx, dy, dz);
                hit = r2 < H2 && (int64_t)j != i;
                extra = hit && !(r2 < pj.w * pj.w);
            }
            const uint32_t hm = (uint32_t)((__ballot(hit) >> gshift) & (((uint64_t)1 << G) - 1));
            if (hit) {
                gidx[first + cg + __popc(hm & below)] = j;
                if (extra) etmp[atomicAdd(&efill[j], 1)] = (int32_t)i;
            }
            cg += __popc(hm);
        }
        // the list is rewritten by the next batch only after every lane read it
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// ---- the first walk: a wavefront per P consecutive particles
//
// Consecutive particles of the sort lie next to one another, so the cells
// about one of them are mostly the cells about all of them. The wavefront
// takes its particles in runs (one box, one level, a small block of cells) and
// lists the cells about the whole run once, 64 cells a step; the concatenated candidates of those cells
// then go 64 at a time, one per lane, past every particle of the run, whose
// position and squared support sit in scalar registers. A candidate is loaded
// and located once for P tests, and a test is the separation, r^2, two
// compares and the ballot that places the hits.
//
// A run's cells are visited in the order of a single particle's walk (z-major,
// then y, then x, particles ascending within a cell, at the same level), and
// the cells that only other particles of the run need hold no hit of this one:
// every row is the list a walk of its own gives, entry for entry.
//
// Bound: vector instruction issue (0.87 instructions a CU and cycle; a loop of
// fused multiply-adds reaches 0.97), then the latency of a batch; seven or eight
// wavefronts per SIMD hide it, hence the register bound. A lognormal box of 128^3 (67 gather partners a particle): a group of
// lanes per particle tested 218 candidates each for 400 vector instructions a
// particle and 1.67 ms; here 370 candidates a particle pass for 255, 1.21 ms
// (64^3: 0.355 to 0.18 ms). Of that, listing only cells in reach of some
// particle of the run took 540 candidates to 370 (1.51 to 1.39 ms), finding a
// candidate's range from head bits instead of a bisection 70 of 105
// instructions a batch (to 1.25 ms), and rows gathered in LDS a wait for their
// stores in every batch (to 1.21 ms).

// cells a run's list may cover, and along one axis at most kAxisCells
constexpr int kRunCells = 216;
// ranges listed at a time
constexpr int kRunRanges = 128;
// 64-candidate batches whose ranges are found by counting head bits
constexpr int kHeadWords = 32;

// inclusive sum over the 64 lanes (DPP row shifts, then the row broadcasts)
__device__ __forceinline__ int wave_incl_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);   // row_shr 1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);   // row_shr 2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);   // row_shr 4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);   // row_shr 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast 15
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // row_bcast 31
    return x;
}

__device__ __forceinline__ double readlane_f64(double x, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                            __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// hits of a row kept in LDS until the wavefront's walk ends (rows seldom
// outgrow them; what does goes straight to the scratch row)
template <int P>
constexpr int kRowSlots = P == 8 ? 96 : P == 4 ? 160 : P == 2 ? 256 : 512;

// LDS of one wavefront of the walk
template <int P>
struct RunLds {
    uint32_t row[P][kRowSlots<P>];
    // squared gap along each axis from particle p to cell e, in cell sides;
    // along x less p's squared support, so that a sum <= 0 means in reach
    __align__(16) float g2[3][kAxisCells][P < 4 ? 4 : P];
    uint64_t head[kHeadWords];                  // bit f set: a range starts at candidate f
    int32_t b[kRunRanges], c[kRunRanges];       // first particle, offset in the concatenation
    uint32_t id[3][kAxisCells];                 // Morton bits and image code, as AxisTab
    uint8_t code[kRunRanges];                   // image shift code
};

// how a run's separations are formed: one image shift per listed cell, all of
// them zero or not, or the minimum-image rule
enum { kNoShift = 0, kShift = 1, kMinImage = 2 };

// one batch of 64 candidates (j, its position and support, in lane order)
// past the wavefront's particles whose bits are set in run; returns how many
// of them the lane's candidate is an extra of
template <int P, int MODE>
__device__ __forceinline__ uint32_t walk_batch(RunLds<P> &s, const double (&X)[P], const double (&Y)[P],
                                               const double (&Z)[P], const double (&H2)[P], uint32_t (&at)[P],
                                               int run, int32_t i0, int32_t j, const double4 &pj, double sx,
                                               double sy, double sz, double L, double hL, int cap,
                                               uint32_t *rows) {
    const double hj2 = pj.w * pj.w;
    uint32_t ne = 0;
    // opaque copies, so that what follows from them per particle is formed
    // anew in each batch: held across the batches it would push the
    // particles' positions out of the scalar registers
    asm volatile("" : "+s"(run), "+s"(cap), "+s"(i0));
    // a batch that holds one of the wavefront's own particles
    const uint64_t own = __builtin_amdgcn_ballot_w64((uint32_t)(j - i0) < (uint32_t)P);
#pragma unroll
    for (int p = 0; p < P; p++) {
        if (!(run >> p & 1)) continue;   // uniform
        double dx, dy, dz;
        if (MODE == kMinImage) {
            dx = min_image(X[p] - pj.x, L, hL);
            dy = min_image(Y[p] - pj.y, L, hL);
            dz = min_image(Z[p] - pj.z, L, hL);
        } else {
            dx = X[p] - pj.x;
            dy = Y[p] - pj.y;
            dz = Z[p] - pj.z;
            if (MODE == kShift) {
                dx += sx;
                dy += sy;
                dz += sz;
            }
        }
        const double r2 = r2_exact(dx, dy, dz);
        uint64_t hm = __builtin_amdgcn_ballot_w64(r2 < H2[p]);
        if (own != 0) hm &= ~__builtin_amdgcn_ballot_w64(j == i0 + p);   // uniform
        if (hm == 0) continue;                                          // uniform
        const uint32_t end = at[p] + __popcll(hm);
        if (__builtin_amdgcn_inverse_ballot_w64(hm)) {
            const uint32_t e = r2 < hj2 ? 0u : 1u, w = (e << 31) | (uint32_t)j;
            const uint32_t k = __builtin_amdgcn_mbcnt_hi((uint32_t)(hm >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)hm, at[p]));
            if (end <= (uint32_t)kRowSlots<P>) {   // uniform
                s.row[p][k] = w;
            } else if (k < (uint32_t)kRowSlots<P>) {
                s.row[p][k] = w;
            } else if (k < (uint32_t)cap) {
                rows[(uint32_t)(p * cap) + k] = w;
            }
            ne += e;
        }
        at[p] = end;
    }
    return ne;
}

// The candidates of the nr listed ranges (cum of them), 64 at a time; the
// next batch's positions load while this one is tested. Loads, stores and
// atomics of a wavefront complete in order, so a wait for the positions is a
// wait for all that was issued before it: hits gather in LDS, and the extras
// of a batch are counted only after the next positions have arrived.
template <int P, int MODE>
__device__ __forceinline__ void walk_list(const double4 *__restrict__ posH, RunLds<P> &s, int nr, int cum,
                                          int lane, const double (&X)[P], const double (&Y)[P],
                                          const double (&Z)[P], const double (&H2)[P], uint32_t (&at)[P],
                                          int run, int32_t i0, double L, double hL, int cap,
                                          uint32_t *rows, int32_t *rcnt, const double (*shifts)[3]) {
    const int top = nr > 1 ? 1 << (31 - __builtin_clz(nr - 1)) : 0;   // largest power of two below nr
    int before = -1;   // range of the candidate before the batch
    auto fetch = [&](int f0, int32_t &j, double4 &pj, int &code) {
        const int f = f0 + lane;
        int r = 0;
        if (f0 < 64 * kHeadWords) {
            // the ranges that start at or before this lane's candidate
            const uint64_t hd = s.head[f0 >> 6];
            const uint32_t h0 = __builtin_amdgcn_readfirstlane((uint32_t)hd),
                           h1 = __builtin_amdgcn_readfirstlane((uint32_t)(hd >> 32));
            r = before + (int)(h0 & 1u) +
                (int)__builtin_amdgcn_mbcnt_hi(h1 >> 1, __builtin_amdgcn_mbcnt_lo(h0 >> 1 | h1 << 31, 0u));
            before += __popc(h0) + __popc(h1);
        } else {
            for (int t = top; t > 0; t >>= 1)
                if (r + t < nr && s.c[r + t] <= f) r += t;
        }
        j = -1;
        code = 0;
        // past the end: at infinity, so no test hits
        pj = make_double4(INFINITY, INFINITY, INFINITY, 0.0);
        if (f < cum) {
            j = s.b[r] + (f - s.c[r]);
            if (MODE == kShift) code = s.code[r];
            pj = posH[(uint32_t)j];
        }
    };
    int32_t jn, jp = 0;
    uint32_t ne = 0;
    double4 pn;
    int cn;
    fetch(0, jn, pn, cn);
    for (int f0 = 0; f0 < cum; f0 += 64) {
        const int32_t j = jn;
        const double4 pj = pn;
        double sx = 0.0, sy = 0.0, sz = 0.0;
        if (MODE == kShift) {
            sx = shifts[cn][0];
            sy = shifts[cn][1];
            sz = shifts[cn][2];
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);   // the positions are here
        __builtin_amdgcn_sched_barrier(0);
        if (ne) atomicAdd(&rcnt[jp], (int)ne);
        if (f0 + 64 < cum) fetch(f0 + 64, jn, pn, cn);
        ne = walk_batch<P, MODE>(s, X, Y, Z, H2, at, run, i0, j, pj, sx, sy, sz, L, hL, cap, rows);
        jp = j;
    }
    if (ne) atomicAdd(&rcnt[jp], (int)ne);
}

template <int P>
__global__ __launch_bounds__(kBlock, P == 8 ? 7 : 8) void k_walk(const double4 *__restrict__ posH, int64_t n, Levels v,
                                                 const int32_t *__restrict__ cbeg,
                                                 const int32_t *__restrict__ cend, int cap, uint32_t *scratch,
                                                 int32_t *ng, int32_t *rcnt, int shift) {
    static_assert(P <= 8, "the axis tables hold eight particles");
    __shared__ double s_shift[27][3];
    __shared__ RunLds<P> s_run[kBlock / 64];
    fill_shifts(s_shift, v.L);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    // the wavefront's number and all that follows from it in scalar registers
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t i0 = (xcd_block(blockIdx.x, gridDim.x) * (kBlock / 64) + wave) * (int64_t)P;
    if (i0 >= n) return;   // whole waves leave together
    RunLds<P> &s = s_run[wave];
    const int np = (int)(n - i0 < P ? n - i0 : P);
    // lane p holds particle p's walk (lanes past the last repeat it)
    const int64_t il = i0 + (lane < np ? lane : np - 1);
    const double4 pl = posH[il];
    const int kl = level_for(pl.w * (double)(1 << shift), v);
    const int bl = (int)(v.skey[il] >> (3 * v.bits));
    // cells of the walk per axis, first + 1024 above the end + 1024; the level
    // with the culling flag above it
    uint32_t rg[3], kc_;
    {
        const int nck = 1 << (v.bits - kl);
        const Grid g{v.L, v.hL, (double)nck / v.L, v.margin, nck};
        int lo, cnt;
        axis_range(pl.x, pl.w, g, lo, cnt);
        rg[0] = (uint32_t)(lo + 1024) << 16 | (uint32_t)(lo + cnt + 1024);
        axis_range(pl.y, pl.w, g, lo, cnt);
        rg[1] = (uint32_t)(lo + 1024) << 16 | (uint32_t)(lo + cnt + 1024);
        axis_range(pl.z, pl.w, g, lo, cnt);
        rg[2] = (uint32_t)(lo + 1024) << 16 | (uint32_t)(lo + cnt + 1024);
        // the support widened by twice the axis margin (far above any rounding)
        kc_ = (uint32_t)kl | (2.0 * ((pl.w + 2.0 * v.margin) + v.L / (double)nck) < v.L ? 256u : 0u);
    }
    double X[P], Y[P], Z[P], H2[P];
    uint32_t at[P];   // hits of each particle so far
    const double hl2 = pl.w * pl.w;
#pragma unroll
    for (int p = 0; p < P; p++) {
        const double4 q = posH[i0 + (p < np ? p : np - 1)];   // uniform: scalar loads
        X[p] = q.x;
        Y[p] = q.y;
        Z[p] = q.z;
        H2[p] = readlane_f64(hl2, p);
        at[p] = 0;
    }
    // particle lane & 7 for the axis tables
    const double px = __shfl(pl.x, lane & 7, 64), py = __shfl(pl.y, lane & 7, 64),
                 pz = __shfl(pl.z, lane & 7, 64), ph = __shfl(pl.w, lane & 7, 64);
    uint32_t *rows = scratch + (size_t)i0 * cap;
    for (int p0 = 0; p0 < np;) {
        // the run p0 .. p1-1: particles of one box and one level whose cells
        // together stay a small block (a step of the sort along the curve can
        // be long; the next run starts there). Without culling the wrapped
        // range decides the order, so it has to be the same for all.
        const uint32_t kc = __builtin_amdgcn_readlane(kc_, p0);
        const int k = (int)(kc & 255u), cull = (int)(kc >> 8), bx = __builtin_amdgcn_readlane(bl, p0);
        int ul[3], uh[3];
#pragma unroll
        for (int a = 0; a < 3; a++) {
            const uint32_t r = __builtin_amdgcn_readlane(rg[a], p0);
            ul[a] = (int)(r >> 16);
            uh[a] = (int)(r & 0xffffu);
        }
        int p1 = p0 + 1;
        while (p1 < np) {
            bool ok = __builtin_amdgcn_readlane(kc_, p1) == kc && __builtin_amdgcn_readlane(bl, p1) == bx;
            int nl[3], nh[3], cells = 1;
#pragma unroll
            for (int a = 0; a < 3; a++) {
                const uint32_t r = __builtin_amdgcn_readlane(rg[a], p1);
                const int l1 = (int)(r >> 16), h1 = (int)(r & 0xffffu);
                nl[a] = l1 < ul[a] ? l1 : ul[a];
                nh[a] = h1 > uh[a] ? h1 : uh[a];
                if (!cull) ok = ok && l1 == ul[a] && h1 == uh[a];
                ok = ok && nh[a] - nl[a] <= kAxisCells;
                cells *= nh[a] - nl[a];
            }
            if (!ok || cells > kRunCells) break;
#pragma unroll
            for (int a = 0; a < 3; a++) {
                ul[a] = nl[a];
                uh[a] = nh[a];
            }
            p1++;
        }
#pragma unroll
        for (int a = 0; a < 3; a++) {
            ul[a] -= 1024;
            uh[a] -= 1024;
        }
        const int nck = 1 << (v.bits - k);
        const double cs = v.L / (double)nck;
        const int mx = uh[0] - ul[0], my = uh[1] - ul[1], mz = uh[2] - ul[2];
        const int ncell = mx * my * mz;
        // axis tables: Morton bits and image code of each cell along an axis;
        // per particle of the run the gap to it, in FP32 with a margin far
        // above its rounding (a cell is listed when it is in reach of any)
        const double ics = (double)nck / v.L;
        if (lane < 3 * kAxisCells) {
            const int a = lane / kAxisCells, e = lane % kAxisCells;
            const int kc = (a == 0 ? ul[0] : a == 1 ? ul[1] : ul[2]) + e;
            const int code = !cull ? 0 : kc < 0 ? 1 : (kc >= nck ? 2 : 0);
            s.id[a][e] = (spread3(wrapc(kc, nck)) << a) | ((uint32_t)code << 30);
        }
        {
            const int e = lane >> 3, p = lane & 7;   // (lanes past P hold no particle)
            const bool in = p >= p0 && p < p1;
            float reach = in ? 1e30f : -1e30f;
            if (cull && in) {
                const float h = (float)((ph + 2.0 * v.margin) * ics);
                reach = h * h * 1.00001f + 1e-5f;
            }
#pragma unroll
            for (int a = 0; a < 3; a++) {
                // the particle from the run's first cell, in cell sides
                const float t = (float)((a == 0 ? px : a == 1 ? py : pz) * ics - (double)ul[a]);
                const float g = fmaxf(0.0f, fmaxf((float)e - t, t - (float)(e + 1)));
                if (p < P) s.g2[a][e][p] = (cull ? g * g : 0.0f) - (a == 0 ? reach : 0.0f);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int32_t *cb = cbeg + (int64_t)bx * v.box_stride + v.off[k];
        const int32_t *ce = cend + (int64_t)bx * v.box_stride + v.off[k];
        const uint32_t dvx = div16(mx), dvy = div16(my);
        const int run = (1 << p1) - (1 << p0);
        for (int c0 = 0; c0 < ncell;) {
            int nr = 0, cum = 0;
            uint64_t shifted = 0;
            if (lane < kHeadWords) s.head[lane] = 0;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            while (c0 < ncell && nr + 64 <= kRunRanges) {
                const int cidx = c0 + lane;
                int jb = 0, len = 0, code = 0;
                if (cidx < ncell) {
                    const int t = (int)(((uint32_t)cidx * dvx) >> 16);
                    const int e = cidx - t * mx;
                    const int a = (int)(((uint32_t)t * dvy) >> 16);
                    const int b = t - a * my;
                    float near = INFINITY;
#pragma unroll
                    for (int p = 0; p < P; p++)
                        near = fminf(near, (s.g2[2][a][p] + s.g2[1][b][p]) + s.g2[0][e][p]);
                    if (near <= 0.0f) {
                        const uint32_t ix = s.id[0][e], iy = s.id[1][b], iz = s.id[2][a];
                        const uint32_t id = (ix | iy | iz) & 0x3fffffffu;
                        code = (int)(ix >> 30) + 3 * (int)(iy >> 30) + 9 * (int)(iz >> 30);
                        jb = cb[id];
                        len = ce[id] - jb;
                    }
                }
                const int inc = wave_incl_scan(len);
                const uint64_t hmk = __builtin_amdgcn_ballot_w64(len > 0);
                if (len > 0) {
                    const int pos = nr + (int)__builtin_amdgcn_mbcnt_hi(
                                             (uint32_t)(hmk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hmk, 0u));
                    s.b[pos] = jb;
                    s.c[pos] = cum + (inc - len);
                    s.code[pos] = (uint8_t)code;
                    const int f = cum + (inc - len);
                    if (f < 64 * kHeadWords) atomicOr((uint32_t *)s.head + (f >> 5), 1u << (f & 31));
                }
                shifted |= __builtin_amdgcn_ballot_w64(len > 0 && code != 0);
                nr += __popcll(hmk);
                cum += __builtin_amdgcn_readlane(inc, 63);
                c0 += 64;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (!cull)
                walk_list<P, kMinImage>(posH, s, nr, cum, lane, X, Y, Z, H2, at, run, (int32_t)i0, v.L, v.hL,
                                        cap, rows, rcnt, s_shift);
            else if (shifted)
                walk_list<P, kShift>(posH, s, nr, cum, lane, X, Y, Z, H2, at, run, (int32_t)i0, v.L, v.hL, cap,
                                     rows, rcnt, s_shift);
            else
                walk_list<P, kNoShift>(posH, s, nr, cum, lane, X, Y, Z, H2, at, run, (int32_t)i0, v.L, v.hL,
                                       cap, rows, rcnt, s_shift);
            // the list is rewritten only after every lane read it
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        p0 = p1;
    }
    // the rows leave LDS 64 entries a store
#pragma unroll
    for (int p = 0; p < P; p++) {
        uint32_t m = at[p] < (uint32_t)kRowSlots<P> ? at[p] : (uint32_t)kRowSlots<P>;
        m = m < (uint32_t)cap ? m : (uint32_t)cap;
        for (uint32_t k = lane; k < m; k += 64) rows[(uint32_t)(p * cap) + k] = s.row[p][k];
    }
    int cnt = 0;
#pragma unroll
    for (int p = 0; p < P; p++)
        if (lane == p) cnt = (int)at[p];
    if (lane < np) ng[i0 + lane] = cnt;
}

// The rows past the scratch rows' slots, walked again straight into place
// (gather row and extras): a grid of any size whose groups of G lanes take the
// particles that compaction listed in longs (longs[0] counts them, the list
// follows) in turn, so it costs nothing when no row is long. The list is short,
// so the blocks go round the XCDs in order.
template <int G>
__global__ __launch_bounds__(kBlock) void k_walk_long(const double4 *__restrict__ posH, Levels v,
                                                      const int32_t *__restrict__ cbeg,
                                                      const int32_t *__restrict__ cend, int cap,
                                                      const int32_t *__restrict__ ng,
                                                      const int64_t *__restrict__ goff, int32_t *gidx,
                                                      int32_t *efill, int32_t *etmp, int shift,
                                                      const int32_t *__restrict__ longs) {
    // the shift table first: every wave of the block is still running
    constexpr int NG = kBlock / G, NR = walk_ranges<G>();
    __shared__ double s_shift[27][3];
    __shared__ int32_t s_b[NG][NR], s_c[NG][NR + 1];
    __shared__ uint8_t s_code[NG][NR];
    __shared__ AxisTab s_ax[NG];
    fill_shifts(s_shift, v.L);
    __syncthreads();
    const int l = threadIdx.x % G, grp = threadIdx.x / G;
    const int gshift = (threadIdx.x & 63) - l;
    const uint32_t below = l == 0 ? 0u : (1u << l) - 1u;
    const int64_t nl = longs[0];
    const int64_t stride = (int64_t)gridDim.x * NG;
    for (int64_t t = (int64_t)blockIdx.x * NG + grp; t < nl; t += stride) {
        const int64_t i = longs[1 + t];
        // a recorded step whose lists overflowed their capacities has its
        // counts cleared: then nothing is written
        if (ng[i] <= cap) continue;
        const double4 pi = posH[i];
        const int k = level_for(pi.w * (double)(1 << shift), v);
        const int nck = 1 << (v.bits - k);
        const Grid g{v.L, v.hL, (double)nck / v.L, v.margin, nck};
        int lx, ly, lz, mx, my, mz;
        axis_range(pi.x, pi.w, g, lx, mx);
        axis_range(pi.y, pi.w, g, ly, my);
        axis_range(pi.z, pi.w, g, lz, mz);
        const int64_t base = box_base(v, i) + v.off[k];
        // the support widened by twice the axis margin (far above any rounding)
        const double cs = v.L / (double)nck;
        const double Hc = pi.w + 2.0 * v.margin;
        if (2.0 * (Hc + cs) < v.L)
            walk_row_flat<G, true>(posH, i, pi, l, gshift, below, v, cbeg + base, cend + base, nck, lx, ly, lz,
                                   mx, my, mz, cs, Hc * Hc, goff[i], gidx, efill, etmp, s_b[grp], s_c[grp],
                                   s_code[grp], s_ax[grp], s_shift);
        else
            walk_row_flat<G, false>(posH, i, pi, l, gshift, below, v, cbeg + base, cend + base, nck, lx, ly, lz,
                                    mx, my, mz, cs, INFINITY, goff[i], gidx, efill, etmp, s_b[grp], s_c[grp],
                                    s_code[grp], s_ax[grp], s_shift);
    }
}

// scratch rows -> gather rows, for rows that fit in cap (G lanes per row
// read and write consecutive slots; longer rows are listed for the second
// walk); each extra (j, i) goes to a slot of row j of the transposed lists
// (efill[j], which the offsets scan set to row j's start, hands out its
// places; slot order is fixed later by rank). A lane takes U entries of its row at
// a time: their loads, then the slot atomics of their extras, then the
// dependent stores, so the atomics' round trips overlap instead of
// following one another.
//
// With VOL, each row's FP64 volume sum of eq. (vol) comes along: W(r_ij, H_i)
// over the self pair and every gather entry, the terms of the volume pass
// (same separations, square root and weight), summed in the order k = l,
// l + G, ... of each lane; n_i goes to vnsum[i] and (x_i, V_i = 1 / n_i) to
// posV[i]. The rows past cap get theirs from k_volume_longs after the second
// walk.
//
// Bound: latency (three quarters of the wavefronts' time is waits) and the
// extras' scattered 4-byte stores. The partners' positions load while the
// atomics are on their way; with the row read again for the volumes once the
// scatter was done, and eight entries at a time, 128^3 took 1.235 ms, three
// entries (68 VGPRs, seven wavefronts a SIMD) 1.056; two 1.043, but 268
// neighbours 0.229 ms against 0.212 (0.25 before). Without volumes eight entries
// (128^3 0.91 ms with three, 0.88; lattice 100^3 with 128 neighbours 0.284 and
// 0.245).
template <int G, int U, bool VOL>
__global__ __launch_bounds__(kBlock) void k_compact_rows(const uint32_t *__restrict__ scratch, int cap,
                                                         int64_t n, const int32_t *__restrict__ ng,
                                                         const int64_t *__restrict__ goff, int32_t *gidx,
                                                         int32_t *efill, int32_t *etmp, int32_t *longs,
                                                         const double4 *__restrict__ posH, Box box,
                                                         double *vnsum, double4 *posV) {
    int64_t gid = xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    const int l = (int)(gid % G);
    const int64_t i = gid / G;
    if (i >= n) return;
    const int cnt = ng[i];
    if (cnt > cap) {
        // walked again into place (the list order is immaterial)
        if (l == 0) longs[1 + atomicAdd(&longs[0], 1)] = (int32_t)i;
        return;
    }
    const uint32_t *row = scratch + (size_t)i * cap;
    const int64_t gw = goff[i];
    double4 pi = make_double4(0.0, 0.0, 0.0, 1.0);
    if (VOL) pi = posH[i];
    const double invH = 1.0 / pi.w;
    const double cw = kW * invH * invH * invH;
    double sum = l == 0 ? cw : 0.0;   // the self pair: W(0, H_i)
    for (int k0 = l; k0 < cnt; k0 += G * U) {
        uint32_t w[U];
#pragma unroll
        for (int u = 0; u < U; u++) w[u] = k0 + u * G < cnt ? row[k0 + u * G] : 0u;
        // the partners' positions are on their way before the stores and atomics
        double4 pj[U];
        if (VOL)
#pragma unroll
            for (int u = 0; u < U; u++) pj[u] = posH[k0 + u * G < cnt ? w[u] & 0x7fffffffu : (uint32_t)i];
        // the returned places are used only after every atomic is issued
        // (efill[j] starts at row j's offset, so the atomic returns the place)
        int32_t at[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int k = k0 + u * G;
            at[u] = -1;
            if (k < cnt) {
                gidx[gw + k] = (int32_t)(w[u] & 0x7fffffffu);
                if (w[u] & 0x80000000u) at[u] = atomicAdd(&efill[(int32_t)(w[u] & 0x7fffffffu)], 1);
            }
        }
        if (VOL)
#pragma unroll
            for (int u = 0; u < U; u++) {
                if (k0 + u * G >= cnt) break;
                const double dx = pair_image(pi.x - pj[u].x, box), dy = pair_image(pi.y - pj[u].y, box),
                             dz = pair_image(pi.z - pj[u].z, box);
                const double q = sqrt_dist(dx * dx + dy * dy + dz * dz) * invH;
                sum += kernel_w(q, cw);
            }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (at[u] >= 0) etmp[at[u]] = (int32_t)i;
    }
    if (VOL) {
#pragma unroll
        for (int m = G / 2; m >= 1; m >>= 1) sum += __shfl_xor(sum, m, G);
        if (l == 0) {
            vnsum[i] = sum;
            posV[i] = make_double4(pi.x, pi.y, pi.z, 1.0 / sum);
        }
    }
}

// The FP64 volume sums of the rows listed in longs (those over the scratch
// rows' cap, written into place by the second walk), as k_compact_rows
// forms them (with its G, lane l adds entries l, l + G, ... and the same
// reduction follows, so the sum is bit for bit the compaction's), over a
// grid of any size.
template <int G>
__global__ __launch_bounds__(kBlock) void k_volume_longs(const int32_t *__restrict__ longs,
                                                         const int32_t *__restrict__ ng, int cap,
                                                         const int64_t *__restrict__ goff,
                                                         const int32_t *__restrict__ gidx,
                                                         const double4 *__restrict__ posH, Box box,
                                                         double *vnsum, double4 *posV) {
    const int64_t gid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int l = (int)(gid % G);
    const int64_t nl = longs[0];
    const int64_t stride = (int64_t)gridDim.x * (kBlock / G);
    for (int64_t t = gid / G; t < nl; t += stride) {
        const int64_t i = longs[1 + t];
        if (ng[i] <= cap) continue;   // cleared by an overflowed recorded step
        const double4 pi = posH[i];
        const double invH = 1.0 / pi.w;
        const double cw = kW * invH * invH * invH;
        double s = l == 0 ? cw : 0.0;
        for (int64_t k = goff[i] + l; k < goff[i + 1]; k += G) {
            const double4 pj = posH[gidx[k]];
            const double dx = pair_image(pi.x - pj.x, box), dy = pair_image(pi.y - pj.y, box),
                         dz = pair_image(pi.z - pj.z, box);
            const double q = sqrt_dist(dx * dx + dy * dy + dz * dz) * invH;
            s += kernel_w(q, cw);
        }
#pragma unroll
        for (int m = G / 2; m >= 1; m >>= 1) s += __shfl_xor(s, m, G);
        if (l == 0) {
            vnsum[i] = s;
            posV[i] = make_double4(pi.x, pi.y, pi.z, 1.0 / s);
        }
    }
}

// Extras rows (per receiving particle j): the walk counts them per j, a
// scan gives the row offsets, the compaction and the second walk drop each
// (j, i) into some slot of row j (atomic slot counters), and here every
// entry moves to the place given by its rank in its row, so each row is
// ascending in i whatever order the slots were taken in. G lanes per row;
// entries of a row are distinct emitters, so the ranks are a permutation of
// the row's slots. A row of up to CAP entries is first staged in LDS (row
// stride CAP + 4 words, so the groups of a wavefront read different banks)
// and every rank is counted from there, four entries per read. Longer rows
// are taken one at a time by the whole wavefront, staged in the LDS of all its
// rows, a tile at a time where they are longer than that (45^3 with 268
// neighbours, a seventh of the rows over 128 entries: 0.73 ms with those
// counted from memory by their own 8 lanes, 0.20 so).
template <int G, int CAP>
__global__ __launch_bounds__(kBlock) void k_extra_rank(const int64_t *__restrict__ eoff,
                                                       const int32_t *__restrict__ tmp, int64_t n,
                                                       int32_t *out, int32_t *eb, int32_t *ee) {
    static_assert(CAP % 4 == 0, "rows are read four entries at a time");
    constexpr int S = CAP + 4, kWave = 64 / G * S;   // words of a row and of a wavefront
    __shared__ __align__(16) int32_t srow[kBlock / 64][kWave];
    const int64_t gid = xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    const int lane = threadIdx.x & 63, l = lane % G;
    int32_t *const sw = srow[threadIdx.x >> 6];
    const int64_t j = gid / G;
    int64_t b = 0;
    int c = 0;
    if (j < n) {
        b = eoff[j];
        c = (int)(eoff[j + 1] - b);
        if (l == 0) {
            eb[j] = (int32_t)b;
            ee[j] = (int32_t)(b + c);
        }
    }
    const auto sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // entries of s below v: m entries, padded to a multiple of four with
    // values above every index
    const auto below = [](const int32_t *s, int m, int32_t v) {
        const int4 *s4 = reinterpret_cast<const int4 *>(s);
        int r = 0;
        for (int u = 0; u < (m + 3) / 4; u++) {
            const int4 q = s4[u];
            r += (q.x < v) + (q.y < v) + (q.z < v) + (q.w < v);
        }
        return r;
    };
    const auto stage = [](int32_t *s, const int32_t *row, int m, int first, int step) {
        for (int t = first; t < ((m + 3) & ~3); t += step) s[t] = t < m ? row[t] : INT32_MAX;
    };
    const bool wide = c > CAP;
    if (!wide) {
        int32_t *sr = sw + lane / G * S;
        stage(sr, tmp + b, c, l, G);
        sync();
        for (int t = l; t < c; t += G) {
            const int32_t v = sr[t];
            out[b + below(sr, c, v)] = v;
        }
    }
    for (uint64_t left = __ballot(wide && l == 0); left; left &= left - 1) {
        const int src = __ffsll((unsigned long long)left) - 1;
        const int64_t bw = __shfl(b, src, 64);
        const int cw = __shfl(c, src, 64);
        for (int t0 = 0; t0 < cw; t0 += 64) {   // an entry a lane
            const int t = t0 + lane;
            const int32_t v = t < cw ? tmp[bw + t] : 0;
            int r = 0;
            for (int s0 = 0; s0 < cw; s0 += kWave) {
                const int m = cw - s0 < kWave ? cw - s0 : kWave;
                if (t0 == 0 || cw > kWave) {   // (a row of one tile is staged once)
                    sync();
                    stage(sw, tmp + bw + s0, m, lane, 64);
                    sync();
                }
                r += below(sw, m, v);
            }
            if (t < cw) out[bw + r] = v;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_set_H(double4 *posH, const double *H, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) posH[i].w = H[i];
}

__global__ __launch_bounds__(kBlock) void k_get_xyz(const double4 *posH, int64_t n, double *x,
                                                    double *y, double *z) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    double4 p = posH[i];
    x[i] = p.x;
    y[i] = p.y;
    z[i] = p.z;
}

__global__ __launch_bounds__(kBlock) void k_permute(const int32_t *perm, const double *src,
                                                    double *dst, int64_t n, int ncomp, int to_sorted) {
    int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= n) return;
    int64_t o = perm[k];
    for (int c = 0; c < ncomp; c++) {
        if (to_sorted) dst[c * n + k] = src[c * n + o];
        else dst[c * n + o] = src[c * n + k];
    }
}

// a step's gas state in sorted order, one launch for all of it (rho and its
// destination may be null)
__global__ __launch_bounds__(kBlock) void k_permute_state(const int32_t *perm, int64_t n, const double *v,
                                                          const double *m, const double *u, const double *rho,
                                                          double *sv, double *sm, double *su, double *srho) {
    int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= n) return;
    int64_t o = perm[k];
    const double a = v[o], b = v[n + o], c = v[2 * n + o], d = m[o], e = u[o], r = rho ? rho[o] : 0.0;
    sv[k] = a;
    sv[n + k] = b;
    sv[2 * n + k] = c;
    sm[k] = d;
    su[k] = e;
    if (rho) srho[k] = r;
}

// row lengths of the exported sets: which 0 -> N_g (self + gather row),
// which 1 -> N_s (gather row + extras row)
__global__ __launch_bounds__(kBlock) void k_export_len(const int64_t *goff, const int32_t *eb,
                                                       const int32_t *ee, int64_t n, int which,
                                                       int64_t *len) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) len[i] = (goff[i + 1] - goff[i]) + (which == 0 ? 1 : (int64_t)(ee[i] - eb[i]));
    if (i == n) len[n] = 0;
}

__global__ __launch_bounds__(kBlock) void k_export_fill(const int64_t *goff, const int32_t *gidx,
                                                        const int32_t *eb, const int32_t *ee,
                                                        const int32_t *eidx, int64_t n, int which,
                                                        const int64_t *off, int32_t *idx) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    int64_t o = off[i];
    if (which == 0) idx[o++] = (int32_t)i;
    for (int64_t k = goff[i]; k < goff[i + 1]; k++) idx[o++] = gidx[k];
    if (which == 1)
        for (int k = eb[i]; k < ee[i]; k++) idx[o++] = eidx[k];
}

inline unsigned nblocks(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

// The input checks: launched, and in an eager build read once they are done.
// boff as in k_validate_final; st in graph mode.
static crk_status launch_checks(crk_ctx *c, const double *x, const double *y, const double *z, const double *H,
                                int64_t n, double L, int64_t *boff, GraphStat *st) {
    const int nblk = (int)std::min<int64_t>((n + kBlock - 1) / kBlock, 1024);
    CRK_TRY(ensure(c, c->red, (size_t)nblk * 3 * sizeof(double) + 64 + (size_t)nblk * sizeof(int)));
    double *part = (double *)c->red.p;
    int *flags = (int *)(part + (size_t)nblk * 3);
    k_validate<<<nblk, kBlock, 0, c->stream>>>(x, y, z, H, n, L, part, flags);
    k_validate_final<<<1, 1024, 0, c->stream>>>(part, flags, nblk, L, boff, n, st ? nullptr : (Checks *)c->pinned.p, st);
    CRK_HIP(c, hipGetLastError());
    if (!st) CRK_HIP(c, hipStreamSynchronize(c->stream));
    return CRK_OK;
}

static crk_status read_checks(crk_ctx *c, double *hmax, double *hmin) {
    const Checks k = *(const Checks *)c->pinned.p;
    *hmax = k.hmax;
    *hmin = k.hmin;
    if (k.flags & 1) return set_err(c, CRK_ERR_NONFINITE, "non-finite position or H");
    if (k.flags & 2) return set_err(c, CRK_ERR_INVALID_ARG, "position outside [0, L)");
    if ((k.flags & 4) || !(*hmin > 0.0)) return set_err(c, CRK_ERR_SUPPORT, "H must be positive");
    return CRK_OK;
}

crk_status validate_inputs(crk_ctx *c, const double *x, const double *y, const double *z,
                           const double *H, int64_t n, double L, double *hmax, double *hmin) {
    CRK_TRY(launch_checks(c, x, y, z, H, n, L, nullptr, nullptr));
    return read_checks(c, hmax, hmin);
}

Levels levels(const crk_ctx *c) {
    Levels v;
    v.L = c->L;
    v.hL = 0.5 * c->L;
    v.c0 = c->cell;
    v.margin = 1e-9 * c->L;
    v.bits = c->bits;
    for (int k = 0; k < 12; k++) v.off[k] = c->lvl_off[k];
    v.skey = (const uint32_t *)c->keyA.p;
    v.box_stride = c->ntab;
    return v;
}

// Particles per wavefront of the walk. More of them share a listed cell and a
// loaded candidate, fewer leave more wavefronts: the device holds 8192 (7168 of
// eight particles), and a wavefront of four particles is worth its half as many
// once it fills that (32^3: 28 us with four, 32 with two and 37 with one;
// 20^3: 57, 45 and 40), one of eight once there are 16 rounds of them, so that
// the last round is a small part (128^3: 1.21 ms with eight, 1.25 with four;
// 64^3: 0.19 and 0.18). The lanes per particle that were asked for bound it.
static int walk_particles(int64_t n, int lanes) {
    const int most = 64 / lanes < 8 ? 64 / lanes : 8;
    int P = n >= (int64_t)8 * 16 * 8192 ? 8 : 4;
    while (P > 1 && (P > most || (P < 8 && n < (int64_t)P * 8192))) P /= 2;
    return P;
}

// Neighbour lists for the current posH / cell tables (cleared: so are the
// walk's counts).
static crk_status build_lists(crk_ctx *c, bool cleared) {
    int64_t n = c->n;
    Levels v = levels(c);
    CRK_TRY(ensure(c, c->ng, (size_t)n * sizeof(int32_t)));
    CRK_TRY(ensure(c, c->goff, (size_t)(n + 1) * sizeof(int64_t)));
    CRK_TRY(ensure(c, c->ecnt, (size_t)n * sizeof(int32_t)));
    CRK_TRY(ensure(c, c->efill, (size_t)n * sizeof(int32_t)));
    CRK_TRY(ensure(c, c->eoff, (size_t)(n + 1) * sizeof(int64_t)));
    int32_t *ng = (int32_t *)c->ng.p;
    int64_t *goff = (int64_t *)c->goff.p;
    int32_t *ecnt = (int32_t *)c->ecnt.p, *efill = (int32_t *)c->efill.p;
    int64_t *eoff = (int64_t *)c->eoff.p;
    const double4 *posH = (const double4 *)c->posH.p;
    const int32_t *cbeg = (const int32_t *)c->cbeg.p, *cend = (const int32_t *)c->cend.p;
    // one walk into a capped scratch row per particle; exact counts come
    // with it, and the extras are counted per receiving particle
    const int cap = std::max(c->walk_cap, c->walk_cap_auto);
    CRK_TRY(ensure(c, c->scratch, (size_t)n * cap * sizeof(uint32_t)));
    uint32_t *scratch = (uint32_t *)c->scratch.p;
    // long rows: longs[0] counts them, their particles follow
    CRK_TRY(ensure(c, c->longs, (size_t)(n + 1) * sizeof(int32_t)));
    int32_t *longs = (int32_t *)c->longs.p;
    if (!cleared) k_zero_counts<<<nblocks(n / 4 + 1), kBlock, 0, c->stream>>>(ecnt, n, longs);
    {
        KTimer kt_(c, "k_walk");
        const int P = walk_particles(n, c->G_walk);
#define L_WALK(PP) k_walk<PP><<<(unsigned)(((n + PP - 1) / PP + kBlock / 64 - 1) / (kBlock / 64)), kBlock, 0, c->stream>>>(posH, n, v, cbeg, cend, cap, scratch, ng, ecnt, c->walk_shift)
        switch (P) {
            case 1: L_WALK(1); break;
            case 2: L_WALK(2); break;
            case 4: L_WALK(4); break;
            default: L_WALK(8); break;
        }
#undef L_WALK
    }
    CRK_HIP(c, hipGetLastError());
    // efill[j] = eoff[j]: the slot counters of the extras rows start at
    // their rows' offsets
    // tot: gather pairs, extra pairs and the longest gather row (for the next
    // build's scratch rows), in graph mode on the device
    CRK_TRY(ensure(c, c->misc, 256));
    int64_t *tot = c->graph_mode ? (int64_t *)c->misc.p + 16 : (int64_t *)c->pinned.p;
    CRK_TRY(scan_counts2(c, ng, ecnt, n, goff, eoff, tot, efill));
    int64_t G, E, longest;
    GraphStat *gst = (GraphStat *)c->gstat.p;
    if (c->graph_mode) {
        // fixed capacities; the counts stay on the device
        G = c->gcap;
        E = c->ecap;
        longest = INT64_MAX;
        k_graph_cap<<<nblocks(n + 1), kBlock, 0, c->stream>>>(tot, G, E, gst, n, goff, eoff, ng);
        CRK_HIP(c, hipGetLastError());
    } else {
        CRK_HIP(c, hipStreamSynchronize(c->stream));
        G = tot[0];
        E = tot[1];
        longest = tot[2];
    }
    if (E > INT32_MAX - 1) return set_err(c, CRK_ERR_INVALID_ARG, "more than 2^31 extra pairs");
    // (four entries more: the passes read whole 16-byte pieces)
    CRK_TRY(ensure(c, c->gidx, (size_t)(G + 4) * sizeof(int32_t)));
    CRK_TRY(ensure(c, c->etmp, (size_t)(E > 0 ? E : 1) * sizeof(int32_t)));
    CRK_TRY(ensure(c, c->eidx, (size_t)(E > 0 ? E : 1) * sizeof(int32_t)));
    CRK_TRY(ensure(c, c->eb, (size_t)n * sizeof(int32_t)));
    CRK_TRY(ensure(c, c->ee, (size_t)n * sizeof(int32_t)));
    int32_t *etmp = (int32_t *)c->etmp.p, *eidx = (int32_t *)c->eidx.p;
    // the FP64 volumes of eq. (vol) come with the compaction when wanted
    const bool vol = c->vol_in_build != 0;
    double *vnsum = nullptr;
    double4 *posV = nullptr;
    if (vol) {
        CRK_TRY(ensure(c, c->vnsum, (size_t)n * sizeof(double)));
        CRK_TRY(ensure(c, c->posV, (size_t)n * sizeof(double4)));
        vnsum = (double *)c->vnsum.p;
        posV = (double4 *)c->posV.p;
    }
    const Box box{c->L, 1.0 / c->L};
    // (the long rows' volumes take the same lanes per row, so a row's sum
    // does not depend on which of the two kernels forms it)
    constexpr int GC = 16;
    {
        KTimer kt_(c, "k_compact_rows");
#define L_COMPACT(U, VOL) k_compact_rows<GC, U, VOL><<<(unsigned)((n * GC + kBlock - 1) / kBlock), kBlock, 0, c->stream>>>(scratch, cap, n, ng, goff, (int32_t *)c->gidx.p, efill, etmp, longs, posH, box, vnsum, posV)
        if (vol) L_COMPACT(3, true);
        else L_COMPACT(8, false);
#undef L_COMPACT
    }
    if (longest > cap) {
        // the rows over the cap are few and long: 32 lanes each (the row is
        // the same list for any lane count), over the list the compaction made
        KTimer kt_(c, "k_walk_long");
        constexpr int GL = 32;
        const unsigned nb = (unsigned)std::min<int64_t>((n * GL + kBlock - 1) / kBlock, 4096);
        k_walk_long<GL><<<nb, kBlock, 0, c->stream>>>(posH, v, cbeg, cend, cap, ng, goff,
                                                      (int32_t *)c->gidx.p, efill, etmp, c->walk_shift, longs);
    }
    CRK_HIP(c, hipGetLastError());
    if (vol && longest > cap) {
        const unsigned nb = (unsigned)std::min<int64_t>((n * GC + kBlock - 1) / kBlock, 1024);
        k_volume_longs<GC><<<nb, kBlock, 0, c->stream>>>(longs, ng, cap, goff, (const int32_t *)c->gidx.p,
                                                          posH, box, vnsum, posV);
        CRK_HIP(c, hipGetLastError());
    }
    // each extras row ascending in the emitting particle
    {
        KTimer kt_(c, "k_extra_rank");
        // longer rows, more lanes and room for each: with 13 extras a particle
        // (128^3) 0.170 ms with 8 lanes and rows of 128, 0.203 with 16 and 256;
        // with 23 (90^3, 96 neighbours) 0.114 both, with 32 0.180 and 0.169; with
        // 75 (45^3, 268 neighbours) 0.204 and 0.111. (In graph mode the last
        // eager build's: the order is the same for both.)
        const double mean = c->graph_mode ? c->mean_extras : (double)E / (double)n;
#define L_RANK(GR, CAP) k_extra_rank<GR, CAP><<<(unsigned)((n * GR + kBlock - 1) / kBlock), kBlock, 0, c->stream>>>(eoff, etmp, n, eidx, (int32_t *)c->eb.p, (int32_t *)c->ee.p)
        if (mean > 32.0) L_RANK(16, 256);
        else L_RANK(8, 128);
#undef L_RANK
    }
    CRK_HIP(c, hipGetLastError());
    if (c->graph_mode) {
        // counts are on the device (crk_graph_replay reads them)
        c->ngather = c->nextra = c->npairs = -1;
    } else {
        c->ngather = G;
        c->mean_extras = (double)E / (double)n;
        c->nextra = E;
        c->npairs = G + E;
        c->walk_cap_auto = walk_cap_next((double)G, (double)n, longest);
    }
    c->built = 1;
    c->have_V = 0;
    c->vol_ready = c->vol_posV = vol ? 1 : 0;
    return CRK_OK;
}

// Steps 2-4 of the build for the geometry held in the context (box offsets
// already on the device). stand_ins: graph mode (see stand_in).
crk_status build_sorted(crk_ctx *c, const double *x, const double *y, const double *z,
                               const double *H, int32_t *perm, bool stand_ins, int64_t *n_pairs,
                               int32_t *n_cells) {
    const int64_t n = c->n;
    const int bits = c->bits;
    const int nboxes = (int)c->nboxes;
    int boxbits = 0;
    while ((1 << boxbits) < nboxes) boxbits++;
    int64_t ntot = c->ntab * nboxes;
    CRK_TRY(ensure(c, c->keyA, (size_t)n * sizeof(uint32_t)));
    CRK_TRY(ensure(c, c->perm, (size_t)n * sizeof(int32_t)));
    uint32_t *key = (uint32_t *)c->keyA.p;
    int32_t *pm = (int32_t *)c->perm.p;
    uint32_t *key_in;
    int32_t *pm_in;
    CRK_TRY(radix_input(c, key, pm, n, 3 * bits + boxbits, &key_in, &pm_in));
    int64_t per_block;
    int32_t *counts;
    CRK_TRY(radix_count(c, n, 3 * bits + boxbits, &per_block, &counts));
    const bool counted = per_block > 0;
    if (!counted) per_block = kBlock;
    k_keys<<<(unsigned)((n + per_block - 1) / per_block), kBlock, 0, c->stream>>>(x, y, z, n, 1.0 / c->cell, c->nc, bits,
                                                  (const int64_t *)(c->graph_mode ? c->gboff.p : c->boff.p),
                                                  nboxes, stand_ins ? H : nullptr, c->L, key_in, pm_in, per_block,
                                                  counted ? counts : nullptr);
    CRK_HIP(c, hipGetLastError());
    {
        KTimer kt_(c, "sort");
        CRK_TRY(radix_sort_pairs(c, key, pm, n, 3 * bits + boxbits, true, counted));
    }
    // 3. sorted particles and the cell tables of every level of every box
    CRK_TRY(ensure(c, c->posH, (size_t)n * sizeof(double4)));
    CRK_TRY(ensure(c, c->cbeg, (size_t)ntot * sizeof(int32_t)));
    CRK_TRY(ensure(c, c->cend, (size_t)ntot * sizeof(int32_t)));
    CRK_TRY(ensure(c, c->ecnt, (size_t)n * sizeof(int32_t)));
    CRK_TRY(ensure(c, c->longs, (size_t)(n + 1) * sizeof(int32_t)));
    k_gather_sorted<<<nblocks(std::max(n, ntot / 4 + 1)), kBlock, 0, c->stream>>>(
        x, y, z, H, pm, n, stand_ins ? 1 : 0, c->L, (double4 *)c->posH.p, perm, (int32_t *)c->cbeg.p,
        (int32_t *)c->cend.p, ntot, (int32_t *)c->ecnt.p, (int32_t *)c->longs.p);
    k_tables<<<nblocks(n), kBlock, 0, c->stream>>>(key, n, levels(c), (int32_t *)c->cbeg.p,
                                                    (int32_t *)c->cend.p);
    CRK_HIP(c, hipGetLastError());
    // 4. neighbour lists
    CRK_TRY(build_lists(c, true));
    if (n_pairs) *n_pairs = c->npairs;
    if (n_cells) *n_cells = c->nc;
    return CRK_OK;
}

crk_status permute_state(crk_ctx *c, const double *v, const double *m, const double *u, const double *rho, double *sv,
                         double *sm, double *su, double *srho) {
    k_permute_state<<<nblocks(c->n), kBlock, 0, c->stream>>>((const int32_t *)c->perm.p, c->n, v, m, u, rho, sv, sm, su,
                                                             srho);
    CRK_HIP(c, hipGetLastError());
    return CRK_OK;
}

}  // namespace crk

using namespace crk;

extern "C" {

crk_status crk_build_cells_batch(crk_ctx *c, int32_t nboxes, const int64_t *box_offsets, int64_t n,
                                 const double *x, const double *y, const double *z, const double *H,
                                 const crk_params *p, double cell_size, int32_t *perm,
                                 int64_t *n_pairs, int32_t *n_cells) {
    if (!c) return CRK_ERR_INVALID_ARG;
    c->singular_clear = 0;
    if (n < 1 || !x || !y || !z || !H || !p || !perm || nboxes < 1 || !box_offsets)
        return set_err(c, CRK_ERR_INVALID_ARG, "crk_build_cells: n < 1 or NULL argument");
    if (n > INT32_MAX / 2) return set_err(c, CRK_ERR_INVALID_ARG, "n too large");
    if (!(p->L > 0.0)) return set_err(c, CRK_ERR_INVALID_ARG, "L must be positive");
    if (box_offsets[0] != 0 || box_offsets[nboxes] != n)
        return set_err(c, CRK_ERR_INVALID_ARG, "box offsets must run from 0 to n");
    for (int b = 0; b < nboxes; b++)
        if (box_offsets[b + 1] < box_offsets[b])
            return set_err(c, CRK_ERR_INVALID_ARG, "box offsets must not decrease");
    CRK_HIP(c, hipSetDevice(c->device));
    const bool gm = c->graph_mode != 0;
    if (gm && (n != c->n || nboxes != c->nboxes || p->L != c->L || !c->built))
        return set_err(c, CRK_ERR_STATE, "graph mode needs the geometry of the last build");
    if (!gm) {
        c->built = 0;
        c->leaf_mode = 0;
        c->nc = 0;
        c->n = n;
        c->L = p->L;
        c->nboxes = nboxes;
    }
    c->have_V = 0;
    c->vol_ready = 0;
    // the FP64 volumes come with the lists unless the pure FP32 mode is asked
    // for (its volume pass sums in FP32)
    c->vol_in_build = p->precision != CRK_MIXED;
    // 1. validate and reduce H
    if (gm) {
        CRK_TRY(ensure(c, c->gstat, sizeof(GraphStat)));
        CRK_TRY(launch_checks(c, x, y, z, H, n, p->L, nullptr, (GraphStat *)c->gstat.p));
        return build_sorted(c, x, y, z, H, perm, true, n_pairs, n_cells);
    }
    CRK_TRY(ensure(c, c->boff, (size_t)(nboxes + 1) * sizeof(int64_t)));
    CRK_TRY(launch_checks(c, x, y, z, H, n, p->L, nboxes == 1 ? (int64_t *)c->boff.p : nullptr, nullptr));
    double hmax = 0.0, hmin = 0.0;
    CRK_TRY(read_checks(c, &hmax, &hmin));
    if (!(hmax < 0.5 * p->L)) return set_err(c, CRK_ERR_SUPPORT, "max H %g >= L/2", hmax);
    // 2. Morton cell hierarchy: finest side near half the smallest support
    //    (or the requested side), at most 256 cells a side and at most about
    //    2^26 table entries over all boxes; box id above the Morton bits
    double cfine = cell_size > 0.0 ? cell_size : 0.5 * hmin;
    int bits = 0;
    while (bits < 8 && p->L / (double)(1 << bits) > cfine &&
           (double)nboxes * (double)((int64_t)1 << (3 * (bits + 1))) * 8.0 / 7.0 <= (double)(1 << 26))
        bits++;
    int boxbits = 0;
    while ((1 << boxbits) < nboxes) boxbits++;
    if (3 * bits + boxbits > 32) return set_err(c, CRK_ERR_INVALID_ARG, "too many boxes for the key width");
    c->bits = bits;
    c->nc = 1 << bits;
    c->cell = p->L / c->nc;
    int64_t off = 0;
    for (int k = 0; k <= bits; k++) {
        c->lvl_off[k] = off;
        int64_t m = (int64_t)1 << (bits - k);
        off += m * m * m;
    }
    c->ntab = off;
    if (nboxes > 1)
        CRK_HIP(c, hipMemcpyAsync(c->boff.p, box_offsets, (size_t)(nboxes + 1) * sizeof(int64_t),
                                  hipMemcpyHostToDevice, c->stream));
    return build_sorted(c, x, y, z, H, perm, false, n_pairs, n_cells);
}

crk_status crk_build_cells(crk_ctx *c, int64_t n, const double *x, const double *y, const double *z,
                           const double *H, const crk_params *p, double cell_size, int32_t *perm,
                           int64_t *n_pairs, int32_t *n_cells) {
    int64_t off[2] = {0, n};
    return crk_build_cells_batch(c, 1, off, n, x, y, z, H, p, cell_size, perm, n_pairs, n_cells);
}

crk_status crk_update_support(crk_ctx *c, const double *H_sorted, int64_t *n_pairs) {
    if (!c) return CRK_ERR_INVALID_ARG;
    if (!H_sorted) return set_err(c, CRK_ERR_INVALID_ARG, "H_sorted is NULL");
    if (c->nc == 0) return set_err(c, CRK_ERR_STATE, "crk_build_cells has not run");
    CRK_HIP(c, hipSetDevice(c->device));
    int64_t n = c->n;
    CRK_TRY(ensure(c, c->scanTmp, (size_t)n * 3 * sizeof(double)));
    double *xs = (double *)c->scanTmp.p;
    k_get_xyz<<<nblocks(n), kBlock, 0, c->stream>>>((const double4 *)c->posH.p, n, xs, xs + n,
                                                     xs + 2 * n);
    CRK_TRY(launch_checks(c, xs, xs + n, xs + 2 * n, H_sorted, n, c->L, nullptr, nullptr));
    const Checks k = *(const Checks *)c->pinned.p;
    if (k.flags & 1) return set_err(c, CRK_ERR_NONFINITE, "non-finite H");
    if ((k.flags & 4) || !(k.hmin > 0.0)) return set_err(c, CRK_ERR_SUPPORT, "H must be positive");
    if (!(k.hmax < 0.5 * c->L)) return set_err(c, CRK_ERR_SUPPORT, "max H %g >= L/2", k.hmax);
    k_set_H<<<nblocks(n), kBlock, 0, c->stream>>>((double4 *)c->posH.p, H_sorted, n);
    CRK_TRY(build_lists(c, false));
    if (n_pairs) *n_pairs = c->npairs;
    return CRK_OK;
}

crk_status crk_permute(crk_ctx *c, const double *src, double *dst, int32_t ncomp, int32_t to_sorted) {
    if (!c) return CRK_ERR_INVALID_ARG;
    if (!src || !dst || ncomp < 1) return set_err(c, CRK_ERR_INVALID_ARG, "crk_permute: bad argument");
    if (c->nc == 0 && !c->leaf_mode) return set_err(c, CRK_ERR_STATE, "crk_build_cells has not run");
    CRK_HIP(c, hipSetDevice(c->device));
    k_permute<<<nblocks(c->n), kBlock, 0, c->stream>>>((const int32_t *)c->perm.p, src, dst, c->n,
                                                        ncomp, to_sorted);
    CRK_HIP(c, hipGetLastError());
    return CRK_OK;
}

crk_status crk_export_neighbors(crk_ctx *c, int32_t which, int64_t *offsets, int32_t *idx,
                                int64_t cap, int64_t *total) {
    if (!c) return CRK_ERR_INVALID_ARG;
    if (!c->built) return set_err(c, CRK_ERR_STATE, "no neighbour lists");
    if (!offsets || !total || (which != 0 && which != 1))
        return set_err(c, CRK_ERR_INVALID_ARG, "crk_export_neighbors: bad argument");
    CRK_HIP(c, hipSetDevice(c->device));
    int64_t n = c->n;
    *total = which == 0 ? c->ngather + n : c->npairs;
    k_export_len<<<nblocks(n + 1), kBlock, 0, c->stream>>>((const int64_t *)c->goff.p,
                                                            (const int32_t *)c->eb.p,
                                                            (const int32_t *)c->ee.p, n, which, offsets);
    CRK_TRY(scan_exclusive_i64(c, offsets, offsets, n + 1));
    if (idx) {
        if (cap < *total) return set_err(c, CRK_ERR_INVALID_ARG, "cap too small");
        k_export_fill<<<nblocks(n), kBlock, 0, c->stream>>>(
            (const int64_t *)c->goff.p, (const int32_t *)c->gidx.p, (const int32_t *)c->eb.p,
            (const int32_t *)c->ee.p, (const int32_t *)c->eidx.p, n, which, offsets, idx);
    }
    CRK_HIP(c, hipGetLastError());
    CRK_HIP(c, hipStreamSynchronize(c->stream));
    return CRK_OK;
}

}  // extern "C"
