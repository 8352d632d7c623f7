// Block ILU(0) set-up and application for the RAS stage, on the local order
// of every subdomain ("Local potential reordering technique", Eq 30-33; RAS
// stage R(A)^-1 of Algorithm 2).
//
// Device design.  ILU(0) and its triangular solves depend only on which end
// of every coupling comes first in the local order, so the rows of each
// subdomain are grouped into levels of the dependency graph (longest-path
// depth); rows of a level are independent.  Inside a row, predecessors and
// successors stay in local order, so every block update happens in the same
// sequence as a sequential ILU(0) in that order and the factors match it.
//
// One workgroup (16 wavefronts) processes one subdomain level by level; a
// wavefront takes a slice of 32 positions of a level, two lanes per position
// (which hold four blocks of the row in registers; rows with more take two
// positions, and only rows with more than eight, well rows, read the rest from
// memory), and the wavefronts take the slices of the subdomain in turn.  A
// slice may run when all slices of the levels before it are done: the
// wavefronts count finished slices in LDS and wait on that count alone, so one
// that has no slice in a level is not held up by it and requests its next data
// meanwhile.  Levels are a latency chain, so nothing a step waits for is
// requested in that step: the static data of a slice (columns, factor blocks,
// right-hand side) and those y values its rows need that were finished by then
// are requested two steps ahead; the rest were finished in the last few levels
// and are read from an LDS ring that holds the results of the most recent
// rows.  Which of these applies to an entry follows from the fixed schedule, so
// the set-up marks it in the entry's column.  One CU streams a subdomain's
// factors at the rate its outstanding L2 misses allow, so helper workgroups of
// the same launch, placed on the subdomain's XCD, read the static data of the
// slices some levels ahead of the sweep into that XCD's L2; the sweep then
// finds them in L2 rather than in HBM (at 2M cells and 16 subdomains an
// application takes 1,122 us without helpers, 762 with 8 each, 754 with 15).
// The gather of the right-hand side into local order and the restricted
// scatter of the result run as separate full-device kernels.
//
// Compiled without floating-point contraction (reproducible block products).
#include <algorithm>
#include <cstring>
#include <tuple>

#include "r2p_impl.h"

constexpr int BS = 256;
constexpr int WG = 1024;               // threads of a subdomain workgroup
constexpr int NWAVE = WG / 64;
// Sweep workgroup: 16 wavefronts of up to 128 VGPRs, two tasks' data in flight
// each; the wavefronts take a subdomain's slices in turn.  (8 wavefronts with
// four tasks each: 883 us per application at 2M cells and 16 subdomains where
// 16 with two took 817; 12 with two, 820.)
template <class T>
struct Sweep {
    static constexpr int wg = 1024;
    static constexpr int ncw = wg / 64;
};
// Sweep: slot pairs per round of a long (well) row; as many as the registers
// left beside two tasks take.
template <class T>
constexpr int LK = sizeof(T) == 4 ? 8 : 2;
constexpr int MAXK = RAS_MAIN / 2;     // entries per lane held in registers (two lanes per row)
constexpr int MAXLEV = 4096;           // levels per subdomain (set-up limit)
constexpr int PROG_STRIDE = 64;        // ints between two sweeps' progress counters
// The sweep's copy of a factor entry's column (local position, < 2^28) carries
// in its top bits where the sweep finds that column's y value:
constexpr int COL_BITS = 28;
constexpr int COL_MASK = (1 << COL_BITS) - 1;
constexpr int F_RING = 0;              // the LDS ring (finished in the last levels)
constexpr int F_PRE = 1;               // loaded from y two steps before the task runs
constexpr int F_SLOW = 2;              // loaded from y when the task runs (rare)
// padding entries are -1: their top bits read as 15

// True when global row h precedes global row g in the local order.
__device__ __forceinline__ bool before(int h, int g, int n, int order, const double *phi) {
    bool hc = h < n, gc = g < n;
    if (hc != gc) return hc;            // cells before wells
    if (!hc || order == R2P_ORDER_NATURAL) return h < g;
    double a = phi[h], b = phi[g];
    return a > b || (a == b && h < g);
}

// ------------------------------------------------------------------ levels
// Longest-path level of every local row, one workgroup per subdomain, by
// Kahn's algorithm in rounds: round t holds exactly the rows whose last
// predecessor was in round t-1, so a row's round is 1 + the deepest round of
// its predecessors (0 for rows without one).  Each row enters the
// subdomain's queue once; the order inside a round depends on scheduling,
// the rounds do not.  The direction of every coupling comes precomputed
// (apred).  When the subdomain has at most LEV_LDS_ROWS rows and no
// in-degree above 255, the in-degrees live in LDS as packed bytes (a 32-bit
// LDS atomic subtracts 1 from one byte; a counter >= 1 never borrows);
// otherwise in global memory.
//
// A round is a chain: the row from the queue, its successors, their counters,
// the queue, a barrier.  The queue's first LEV_Q rows sit in LDS, and up to
// four successors come as one 16-byte word (SUCC_MORE in it: the row has more,
// see its couplings).  16 subdomains of 135,000 rows in 487 levels: 1.75 ms
// beside the AMG set-up; 4.2 to 5.1 with the couplings looked up through aptr,
// adj and apred and the queue in memory; 2.07 with the words of the rows just
// counted down requested ahead.
constexpr int LEV_LDS_WORDS = 38912;              // 152 KiB of packed counters
constexpr int LEV_LDS_ROWS = 4 * LEV_LDS_WORDS;
constexpr int LEV_Q = 1008;
constexpr int SUCC_MORE = -2;
__global__ __launch_bounds__(WG) void k_levels(const int *suboff, const int *aptr, const int *adj,
                                               const unsigned char *apred, const int4 *succ4,
                                               const int *npred, int *indeg, int *queue, int *lev,
                                               int *nlev) {
    __shared__ unsigned cnt[LEV_LDS_WORDS];
    __shared__ int lq[2][LEV_Q], tail[3], maxd;
    int sub = blockIdx.x;
    int a = suboff[sub], b = suboff[sub + 1];
    if (threadIdx.x == 0) { tail[0] = tail[1] = tail[2] = 0; maxd = 0; }
    __syncthreads();
    int md = 0;
    for (int l = a + (int)threadIdx.x; l < b; l += WG) md = max(md, npred[l]);
    atomicMax(&maxd, md);
    __syncthreads();
    const bool in_lds = b - a <= LEV_LDS_ROWS && maxd <= 255;
    if (in_lds) {
        for (int w = threadIdx.x; w < (b - a + 3) / 4; w += WG) {
            unsigned v = 0;
            for (int k = 0; k < 4; k++) {
                int l = a + 4 * w + k;
                if (l < b) v |= (unsigned)npred[l] << (8 * k);
            }
            cnt[w] = v;
        }
    }
    // the rows of round t are entries 0 .. tail[t mod 3] of its queue: in
    // lq[t & 1], past LEV_Q in queue[] behind those of the rounds before
    int qs = a;
    auto push = [&](int t, int base, int h) {
        int k = atomicAdd(&tail[t % 3], 1);
        if (k < LEV_Q) lq[t & 1][k] = h;
        else queue[base + k] = h;
    };
    for (int l = a + (int)threadIdx.x; l < b; l += WG) {
        int d = npred[l];
        if (!in_lds) indeg[l] = d;
        if (d == 0) push(0, qs, l);
    }
    __syncthreads();
    auto count_down = [&](int h) {           // true for the last predecessor
        if (!in_lds) return atomicSub(&indeg[h], 1) == 1;
        int r = h - a, sh = 8 * (r & 3);
        return ((atomicSub(&cnt[r >> 2], 1u << sh) >> sh) & 255u) == 1u;
    };
    int t = 0;
    for (int n = tail[0]; n > 0;) {
        if (threadIdx.x == 0) tail[(t + 2) % 3] = 0;
        for (int q = threadIdx.x; q < n; q += WG) {
            int l = q < LEV_Q ? lq[t & 1][q] : queue[qs + q];
            lev[l] = t;
            int4 s = succ4[l];
            if (s.x == SUCC_MORE) {
                for (int e = aptr[l]; e < aptr[l + 1]; e++)
                    if (!apred[e] && count_down(adj[e])) push(t + 1, qs + n, adj[e]);
                continue;
            }
            int h[4] = {s.x, s.y, s.z, s.w};
            bool last[4];
            if (in_lds) {
                unsigned old[4];
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    // a missing successor: nothing off the row's own counter
                    int r = (h[k] >= 0 ? h[k] : l) - a;
                    old[k] = atomicSub(&cnt[r >> 2], h[k] >= 0 ? 1u << (8 * (r & 3)) : 0u);
                }
#pragma unroll
                for (int k = 0; k < 4; k++)
                    last[k] = h[k] >= 0 && ((old[k] >> (8 * ((h[k] - a) & 3))) & 255u) == 1u;
            } else {
#pragma unroll
                for (int k = 0; k < 4; k++) last[k] = h[k] >= 0 && count_down(h[k]);
            }
#pragma unroll
            for (int k = 0; k < 4; k++)
                if (last[k]) push(t + 1, qs + n, h[k]);
        }
        __syncthreads();
        qs += n;
        t++;
        n = tail[t % 3];
    }
    if (threadIdx.x == 0) nlev[sub] = t;
}

// Predecessors and successors of every row, the direction of its couplings,
// and its successors as one word (see k_levels).
__global__ void k_pred_count(int mtot, int n, int order, const double *phi, const int *glob_nat,
                             const int *aptr, const int *adj, unsigned char *apred, int *nl,
                             int *nu, int4 *succ4) {
    int l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= mtot) return;
    int g = glob_nat[l], a = 0, c = 0;
    int4 s = make_int4(-1, -1, -1, -1);
    for (int e = aptr[l]; e < aptr[l + 1]; e++) {
        int h = adj[e];
        bool p = before(glob_nat[h], g, n, order, phi);
        apred[e] = p;
        a += p;
        if (!p) {
            s.x = c == 0 ? h : s.x;
            s.y = c == 1 ? h : s.y;
            s.z = c == 2 ? h : s.z;
            s.w = c == 3 ? h : s.w;
            c++;
        }
    }
    if (c > 4) s.x = SUCC_MORE;
    nl[l] = a;
    nu[l] = c;
    succ4[l] = s;
}

// A row that takes two positions.
__device__ __forceinline__ bool is_long(int nl, int nu) { return max(nl, nu) > RAS_MAIN; }

__global__ void k_level_count(int mtot, const int *sub_of, const int *lev, const int *lbase,
                              const int *nl, const int *nu, int *cnt, int *nlong) {
    int l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= mtot) return;
    int seg = lbase[sub_of[l]] + lev[l];
    atomicAdd(&cnt[seg], 1);
    if (is_long(nl[l], nu[l])) atomicAdd(&nlong[seg], 1);
}

// Sort key of a row: its level segment, then long rows, those long in L (key 0)
// before those long in U only (1), then the others in descending predecessor
// count; the sort is stable, rows with equal keys stay in natural local order.
// So the rows of a slice have about as many entries each, and the sweep reads
// only the parts of a slice that some row of it has (2M cells, random pressure,
// where 57% of the rows are long in L or in U, 256 subdomains: 346 us, 380 with
// every part read).
__global__ void k_order_keys(int mtot, const int *sub_of, const int *lev, const int *lbase,
                             const int *nl, const int *nu, unsigned *key, unsigned *val) {
    int l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= mtot) return;
    unsigned seg = (unsigned)(lbase[sub_of[l]] + lev[l]);
    unsigned w = is_long(nl[l], nu[l]) ? nl[l] <= RAS_MAIN : (unsigned)(RAS_MAIN + 2 - nl[l]);
    key[l] = (seg << 3) | w;
    val[l] = (unsigned)l;
}

// Positions of the sorted rows (key: segment << 3 | ..): slices of RAS_ROWS
// positions per level, a level's first slice at soff; two positions per long
// row.
__global__ void k_perm_gather(int mtot, const unsigned *key, const unsigned *perm, const int *lptr,
                              const int *nlong, const int *soff, const int *glob_nat,
                              const unsigned char *owned_nat,
                              const int *nlnat, const int *nunat, const int *dsrc_nat, int *pos,
                              int *permi, int *glob, unsigned char *owned, int *nl, int *nu,
                              int *dsrc) {
    int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= mtot) return;
    int l = (int)perm[q], seg = (int)(key[q] >> 3);
    int i = q - lptr[seg];
    int p = RAS_ROWS * soff[seg] + i + min(i, nlong[seg]);
    permi[p] = l;
    pos[l] = p;
    glob[p] = glob_nat[l];
    owned[p] = owned_nat[l];
    nl[p] = nlnat[l];
    nu[p] = nunat[l];
    dsrc[p] = dsrc_nat[l];
}

__global__ void k_slice_count(int nseg, const int *lptr, const int *nlong, int *nsl) {
    int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g < nseg) nsl[g] = (lptr[g + 1] - lptr[g] + nlong[g] + RAS_ROWS - 1) / RAS_ROWS;
    if (g == nseg) nsl[g] = 0;
}

// Entries of every slice's longest L and U part, its long rows, and the
// overflow entries beyond the main ones; 32 lanes per slice.
__global__ void k_slice_width(int nslice, const int *nl, const int *nu, int *wl, int *wu,
                              int *wlong, int *xl, int *xu) {
    int p = blockIdx.x * blockDim.x + threadIdx.x, sl = p / RAS_ROWS;
    if (p == 0) xl[nslice] = xu[nslice] = 0;
    if (sl >= nslice) return;
    int ml = nl[p], mu = nu[p], lg = is_long(ml, mu);
    for (int d = 1; d < RAS_ROWS; d <<= 1) {
        ml = max(ml, __shfl_xor(ml, d, 64));
        mu = max(mu, __shfl_xor(mu, d, 64));
        lg += __shfl_xor(lg, d, 64);
    }
    if (p % RAS_ROWS) return;
    wl[sl] = ml;
    wu[sl] = mu;
    wlong[sl] = lg;
    xl[sl] = max(0, (ml + 1) / 2 - RAS_MAIN) * RAS_SLICE;
    xu[sl] = max(0, (mu + 1) / 2 - RAS_MAIN) * RAS_SLICE;
}

// Scanned overflow offsets to the starts that RasRow expects.
__global__ void k_overflow_base(int nslice, int *xl, int *xu) {
    int sl = blockIdx.x * blockDim.x + threadIdx.x;
    if (sl >= nslice) return;
    xl[sl] += (nslice - 2) * RAS_MENT;
    xu[sl] += (nslice - 2) * RAS_MENT;
}

// Entries of position p in its slice: predecessors and successors, each in
// ascending local order (insertion sort over the strided slots).
__device__ __forceinline__ void fill_row_long(int p, int n, int order, const double *phi, const int *permi,
                              const int *glob_nat, const int *aptr, const int *adj,
                              const int *asrc, const int *pos, const int *glob, const int *xlb,
                              const int *xub, int *lcol, int *lsrc, int *ucol, int *usrc) {
    int l = permi[p], g = glob_nat[l];
    const RasRow rl(xlb, p), ru(xub, p);
    int el = 0, eu = 0;
    for (int t = aptr[l]; t < aptr[l + 1]; t++) {
        int h = adj[t];
        int gh = glob_nat[h];
        if (before(gh, g, n, order, phi)) {
            long k = rl(el++);
            lcol[k] = pos[h];
            lsrc[k] = asrc[t];
        } else {
            long k = ru(eu++);
            ucol[k] = pos[h];
            usrc[k] = asrc[t];
        }
    }
    for (int part = 0; part < 2; part++) {
        int cnt = part == 0 ? el : eu;
        const RasRow &at = part == 0 ? rl : ru;
        int *col = part == 0 ? lcol : ucol;
        int *src = part == 0 ? lsrc : usrc;
        for (int u = 1; u < cnt; u++) {
            long ku = at(u);
            int vc = col[ku], vs = src[ku];
            int vg = glob[vc];
            int k = u - 1;
            while (k >= 0 && before(vg, glob[col[at(k)]], n, order, phi)) {
                col[at(k + 1)] = col[at(k)];
                src[at(k + 1)] = src[at(k)];
                k--;
            }
            col[at(k + 1)] = vc;
            src[at(k + 1)] = vs;
        }
    }
}

// Placement of every local row's couplings into its L (predecessors) and U
// (successors) entries, each part ascending in the local order.  A row with
// at most FE couplings (every cell row) sorts them in registers: the local
// order is a strict total order on global rows, so sorting all couplings at
// once puts the predecessors first, both parts ascending, and the result is
// the same as the per-part insertion sort that longer rows (wells) use.
constexpr int FE = 8;

// before() on values already loaded: cells ahead of wells, cells by
// decreasing potential then index, wells (or the natural order) by index.
__device__ __forceinline__ bool before_v(int h, double ph, int g, double pg, int n, int order) {
    bool hc = h < n, gc = g < n;
    if (hc != gc) return hc;
    if (!hc || order == R2P_ORDER_NATURAL) return h < g;
    return ph > pg || (ph == pg && h < g);
}

__global__ void k_fill_entries(int npos, int n, int order, const double *phi, const int *permi,
                               const int *glob_nat, const int *aptr, const int *adj,
                               const int *asrc, const int *pos, const int *glob, const int *xlb,
                               const int *xub, int *lcol, int *lsrc, int *ucol, int *usrc) {
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npos) return;
    int l = permi[p];
    if (l < 0) return;
    int t0 = aptr[l], deg = aptr[l + 1] - t0;
    if (deg > FE) {
        fill_row_long(p, n, order, phi, permi, glob_nat, aptr, adj, asrc, pos, glob, xlb, xub, lcol,
                      lsrc, ucol, usrc);
        return;
    }
    const bool pot = order != R2P_ORDER_NATURAL;
    int g = glob_nat[l];
    double pg = (pot && g < n) ? phi[g] : 0.0;
    // INT_MAX pads the unused slots: it sorts after every row
    int gh[FE], ps[FE], sr[FE];
    double pv[FE];
#pragma unroll
    for (int k = 0; k < FE; k++) {
        gh[k] = 0x7fffffff; ps[k] = 0; sr[k] = 0; pv[k] = 0.0;
        if (k < deg) {
            int h = adj[t0 + k];
            gh[k] = glob_nat[h];
            ps[k] = pos[h];
            sr[k] = asrc[t0 + k];
        }
    }
#pragma unroll
    for (int k = 0; k < FE; k++)
        if (pot && gh[k] < n) pv[k] = phi[gh[k]];
    // odd-even transposition sort (FE rounds sort FE keys)
#pragma unroll
    for (int rd = 0; rd < FE; rd++) {
#pragma unroll
        for (int k = rd & 1; k + 1 < FE; k += 2) {
            if (before_v(gh[k + 1], pv[k + 1], gh[k], pv[k], n, order)) {
                int ti = gh[k]; gh[k] = gh[k + 1]; gh[k + 1] = ti;
                ti = ps[k]; ps[k] = ps[k + 1]; ps[k + 1] = ti;
                ti = sr[k]; sr[k] = sr[k + 1]; sr[k + 1] = ti;
                double td = pv[k]; pv[k] = pv[k + 1]; pv[k + 1] = td;
            }
        }
    }
    const RasRow rl(xlb, p), ru(xub, p);
    int el = 0, eu = 0;
#pragma unroll
    for (int k = 0; k < FE; k++) {
        if (k < deg) {
            if (before_v(gh[k], pv[k], g, pg, n, order)) {
                long e = rl(el++);
                lcol[e] = ps[k];
                lsrc[e] = sr[k];
            } else {
                long e = ru(eu++);
                ucol[e] = ps[k];
                usrc[e] = sr[k];
            }
        }
    }
}

// ---------------------------------------------------------- factorisation
// Block ILU(0) in IKJ form: for every predecessor q of row p, in local
// order, L_pq = A_pq U_qq^-1, then A_pj -= L_pq U_qj for every later entry j
// of row p that row q also holds.  The set-up splits this into
//   1. a gather of every row's blocks into the factor arrays (all rows at
//      once; the diagonal block goes where its inverse will be stored);
//   2. a symbolic pass (all rows at once) that finds, for each L entry
//      (p, q), where U_qp sits in row q, plus the rarer matches of other
//      later entries (they need a triangle p-q-j, which the 7-point grid
//      graph does not have; well couplings make them);
//   3. the numeric pass, one workgroup per subdomain, level by level, which
//      only follows the precomputed matches.
// The updates of every target happen in the same order as in the plain
// loop, with the same expressions, so the factors are the same.
struct FactArgs {
    BlkSrc B;
    int npos, n, nx, nxy;
    const int *cell_perf;
    const int *lbase, *nlev, *soff;
    const int *xlb, *xub, *glob;
    const int *nl, *nu, *dsrc, *lcol, *ucol, *lsrc, *usrc;
    int *ldiag;                  // per L entry: entry of U_qp in row q, or -2: it stays A_qp, see tval
    int *xptr;                   // npos+1: first extra match of every position
    int4 *xl;                    // extra matches: (e, e2, entry index in row q's U, 0)
    double *lval, *uval, *dinv;
    double *tval;                // per L entry (p, q): A_qp
    int *status;
    int *prog;                   // as in SweepArgs, zeroed by k_bilu_gather
    int ns, nsp, nhelp;          // as in SweepArgs
};

// Block k of a factor array.
__device__ __forceinline__ void ld_blk(double *v, const double *arr, long k) {
    const double2 a = *(const double2 *)&arr[ras_val(k, 0)],
                  b = *(const double2 *)&arr[ras_val(k, 1)];
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
}
__device__ __forceinline__ void st_blk(double *arr, long k, const double *v) {
    *(double2 *)&arr[ras_val(k, 0)] = make_double2(v[0], v[1]);
    *(double2 *)&arr[ras_val(k, 1)] = make_double2(v[2], v[3]);
}

// Every row's blocks.  U entries change only by extra matches, which wells and
// perforated cells have: for another row q, U_qp of an L entry (p, q) is A_qp
// for good, and is put beside A_pq.  The factorisation then reads it with the
// row's own data, where following ldiag costs two lines of row q.
__global__ void k_bilu_gather(FactArgs A) {
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < A.ns) A.prog[PROG_STRIDE * p] = 0;
    if (p >= A.npos || A.glob[p] < 0) return;
    int nlp = A.nl[p], nup = A.nu[p];
    const RasRow rl(A.xlb, p), ru(A.xub, p);
    double v[4];
    for (int e = 0; e < nlp; e++) {
        const long k = rl(e);
        const int src = A.lsrc[k];
        load_block(A.B, src, v);
        st_blk(A.lval, k, v);
        if (src < 0) continue;
        const int sl = src / A.n;                 // 1 .. 6: a cell's neighbour
        const int q = src - sl * A.n + slot_offset(sl, A.nx, A.nxy);
        if (A.cell_perf[q] >= 0) continue;
        load_block(A.B, ((sl - 1) ^ 1) * A.n + A.n + q, v);
        st_blk(A.tval, k, v);
        A.ldiag[k] = -2;
    }
    for (int e = 0; e < nup; e++) {
        load_block(A.B, A.usrc[ru(e)], v);
        st_blk(A.uval, ru(e), v);
    }
    load_block(A.B, A.dsrc[p], &A.dinv[4 * (long)p]);
}

// Where U_qp sits in row q, for the L entries (p, q) that need it, and the matches of other
// later entries.  Those need a triangle p - q - j, so p is a well or a
// perforated cell (the 7-point grid has none): such positions go on a list
// for k_bilu_sym_well.
__global__ void k_bilu_sym(FactArgs A, int *list, int *nlist) {
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= A.npos) return;
    const int g = A.glob[p];
    if (g >= 0 && (g >= A.n || A.cell_perf[g] >= 0)) {
        list[atomicAdd(nlist, 1)] = p;
        return;
    }
    A.xptr[p] = 0;
    if (g < 0) return;
    const int nlp = A.nl[p];
    const RasRow rl(A.xlb, p);
    for (int e = 0; e < nlp; e++) {
        if (A.ldiag[rl(e)] == -2) continue;
        int qe = A.lcol[rl(e)];
        const RasRow rq(A.xub, qe);
        for (int yy = 0; yy < A.nu[qe]; yy++)
            if (A.ucol[rq(yy)] == p) A.ldiag[rl(e)] = (int)rq(yy);
    }
}

// The listed positions, a wavefront each: pass 0 counts a position's extra
// matches and records the diagonal match of its L entries; pass 1 writes the
// extra matches, by L entry, then by later entry.  The lanes hold the row's
// entries in order (L columns, p itself, U columns), 64 at a time.
__global__ __launch_bounds__(256) void k_bilu_sym_well(FactArgs A, const int *list, const int *nlist,
                                                       int pass) {
    const int lane = threadIdx.x & 63, n = *nlist;
    for (int i = blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += gridDim.x * 4) {
        const int p = __builtin_amdgcn_readfirstlane(list[i]);
        const int nlp = A.nl[p], tot = nlp + A.nu[p];
        const RasRow rl(A.xlb, p), ru(A.xub, p);
        auto entry = [&](int e) {
            return e < nlp ? A.lcol[rl(e)] : (e == nlp ? p : (e <= tot ? A.ucol[ru(e - nlp - 1)] : -9));
        };
        const int c0 = entry(lane), nu0 = lane < nlp ? A.nu[c0] : 0;
        int cnt = 0, out = pass ? A.xptr[p] : 0;
        for (int e = 0; e < nlp; e++) {
            const int q = e < 64 ? __shfl(c0, e, 64) : A.lcol[rl(e)];
            const int nuq = e < 64 ? __shfl(nu0, e, 64) : A.nu[q];
            const RasRow rq(A.xub, q);
            for (int b = (e + 1) & ~63; b <= tot; b += 64) {
                const int e2 = b + lane, cj = b == 0 ? c0 : entry(e2);
                int y = -1;
                for (int yb = 0; yb < nuq; yb += 64) {
                    int uc = yb + lane < nuq ? A.ucol[rq(yb + lane)] : -2;
                    for (int j = 0; j < min(64, nuq - yb); j++)
                        if (__shfl(uc, j, 64) == cj && y < 0) y = yb + j;
                }
                bool found = y >= 0 && e2 > e && e2 <= tot;
                if (found && e2 == nlp && pass == 0) A.ldiag[rl(e)] = (int)rq(y);
                bool ext = found && e2 != nlp;
                unsigned long long m = __ballot(ext);
                if (pass && ext)
                    A.xl[out + cnt + __popcll(m & ((1ull << lane) - 1))] = make_int4(e, e2, (int)rq(y), 0);
                cnt += __popcll(m);
            }
        }
        if (pass == 0 && lane == 0) A.xptr[p] = cnt;
    }
}

__device__ __forceinline__ void mul_blk(double *l, const double *a, const double *dk) {
    l[0] = a[0] * dk[0] + a[1] * dk[2];
    l[1] = a[0] * dk[1] + a[1] * dk[3];
    l[2] = a[2] * dk[0] + a[3] * dk[2];
    l[3] = a[2] * dk[1] + a[3] * dk[3];
}

__device__ __forceinline__ void sub_prod(double *t, const double *l, const double *u) {
    t[0] -= l[0] * u[0] + l[1] * u[2];
    t[1] -= l[0] * u[1] + l[1] * u[3];
    t[2] -= l[2] * u[0] + l[3] * u[2];
    t[3] -= l[2] * u[1] + l[3] * u[3];
}

// t -= l u for blocks of the factor arrays.
__device__ __forceinline__ void sub_prod_at(double *tarr, long kt, const double *l,
                                            const double *uarr, long ku) {
    double t[4], u[4];
    ld_blk(t, tarr, kt);
    ld_blk(u, uarr, ku);
    sub_prod(t, l, u);
    st_blk(tarr, kt, t);
}

// L entry e of row p (block a = A_pq, pivot dk = D_q^-1, ud = U_qp unless kd =
// -1): the multiplier l = A_pq D_q^-1 replaces A_pq, then every later entry of
// row p that row q's U part reaches loses l times that U block, in the row's
// order (the remaining L entries, the diagonal, the U entries).
__device__ __forceinline__ void bilu_entry(const FactArgs &A, const RasRow &rl, const RasRow &ru,
                                           int nlp, int e, const double *a, const double *dk, int kd,
                                           const double *ud, double *d, int &xi, int xe) {
    double l[4];
    mul_blk(l, a, dk);
    st_blk(A.lval, rl(e), l);
    for (; xi < xe; xi++) {
        int4 m = A.xl[xi];
        if (m.x != e || m.y > nlp) break;
        sub_prod_at(A.lval, rl(m.y), l, A.uval, m.z);
    }
    if (kd != -1) sub_prod(d, l, ud);
    for (; xi < xe; xi++) {
        int4 m = A.xl[xi];
        if (m.x != e) break;
        sub_prod_at(A.uval, ru(m.y - nlp - 1), l, A.uval, m.z);
    }
}

__device__ __forceinline__ void ld4(double *v, const double *p) {
    const double2 a = ((const double2 *)p)[0], b = ((const double2 *)p)[1];
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
}

// The wavefronts take the subdomain's slices in turn, two lanes per position as
// in the sweep, and a slice runs once the slices of all levels before it are
// finished (a count in LDS; a wavefront waits for slices before its own only, so
// the lowest unfinished one always runs).  A row's own data, which no other row
// changes (its main L blocks, their columns, U_qp blocks and slots, its
// diagonal block), are requested while the wavefront's slice before it is worked
// on, in whole contiguous loads; the slice then waits for the count and for the
// pivots of the rows it names.  Lane 2r + h works on entries h and 2 + h and on
// row h of the diagonal block; the partner's products come by DPP and are
// subtracted in the order of the entries, a long row's second position's after
// its own.  Rows with extra matches or still more entries are worked on by their
// first lane alone, which loads what it needs in turn.
// What bounds it: one CU reads and writes a subdomain's factors, about 61 MB at
// 143,000 positions, with two slices' data in flight per wavefront, so what a
// load takes; helper workgroups on the XCD read ahead into its L2 as for the
// sweep.  16 such subdomains beside the AMG set-up: 3.0 to 3.7 ms with a lane per
// row and a barrier per level; 3.1 in this form with long rows left to one lane,
// 2.5 with them, 2.04 with 4 helpers each (2: 2.27; 8: 2.05; 32 slices ahead
// instead of 64: 2.30).  2,000 cells: 100 us before, 53 now.  16 wavefronts of
// 128 registers spill (5.7 ms), 8 take 2.56 ms without helpers.
constexpr int LPF = 4;
static_assert(LPF == RAS_MAIN, "the main entries are held in registers");
constexpr int BWG = 768;
constexpr int BNW = BWG / 64;

struct BiluRow {
    int p, glob, nlp, xi, xe;     // glob < 0: no row
    int q[2], kd[2];              // entries h, 2 + h
    double2 a0[2], u0[2];         // blocks of entry h: row h, row 1 - h
    double2 a1[2], u1[2];         // rows h of the blocks of entries 2 and 3
    double2 d;                    // row h
};

// No branches, so that the waits stay exact: positions without a row have no
// entries.
__device__ __forceinline__ void bilu_load(const FactArgs &A, BiluRow &R, int sl, int lane) {
    const int p = RAS_ROWS * sl + (lane >> 1);
    R.p = p;
    R.glob = A.glob[p];
    R.nlp = A.nl[p];
    R.xi = A.xptr[p];
    R.xe = A.xptr[p + 1];
    const long k = (long)sl * RAS_MENT + lane;     // entry h; 64 further: entry 2 + h
    const double2 *lv = (const double2 *)A.lval + 2 * (long)sl * RAS_MENT + lane;
    const double2 *tv = (const double2 *)A.tval + 2 * (long)sl * RAS_MENT + lane;
#pragma unroll
    for (int i = 0; i < 2; i++) {
        R.q[i] = A.lcol[k + 64 * i];
        R.kd[i] = A.ldiag[k + 64 * i];
        R.a0[i] = lv[64 * i];
        R.u0[i] = tv[64 * i];
        R.a1[i] = lv[128 + 64 * i];
        R.u1[i] = tv[128 + 64 * i];
    }
    R.d = ((const double2 *)A.dinv)[(long)sl * 64 + lane];
}

__device__ __forceinline__ double2 sel2(bool c, double2 x, double2 y) {
    return make_double2(c ? x.x : y.x, c ? x.y : y.y);
}

// Product of the block row l with block u given as its rows h and 1 - h.
__device__ __forceinline__ double2 row_prod(double2 l, double2 uh, double2 uo, bool h) {
    double x = h ? l.y : l.x, y = h ? l.x : l.y;       // (a sum of two commutes)
    return make_double2(x * uh.x + y * uo.x, x * uh.y + y * uo.y);
}

constexpr int PSPIN = 1 << 16;    // bound of a helper's wait for its subdomain
// Read one dword of every 128-byte line of N ranges, together, so that a chunk
// costs one trip to memory; the values are summed only so that the loads stay.
// The ranges lie in allocations aligned to a line, so the line of a range's
// first byte starts inside its allocation.
template <int N>
struct Lines {
    const char *p[N];
    int n[N];
    __device__ __forceinline__ void set(int k, const void *q, long bytes) {
        p[k] = (const char *)((unsigned long)q & ~127ul);
        n[k] = (int)(((const char *)q + bytes - 1 - p[k]) / 128) + 1;
    }
    __device__ __forceinline__ unsigned touch() const {
        int total = 0;
#pragma unroll
        for (int k = 0; k < N; k++) total += n[k];
        unsigned acc = 0;
        for (int i = threadIdx.x; i < total; i += blockDim.x) {
            const char *a = p[0] + 128l * i;
            int r = i;
#pragma unroll
            for (int k = 0; k + 1 < N; k++)
                if (r >= n[k]) {
                    r -= n[k];
                    a = p[k + 1] + 128l * r;
                } else {
                    r = -1;          // found: below every later count
                }
            acc += *(const unsigned *)a;
        }
        return acc;
    }
};

// A helper's wait before it reads slices i0 .. i0 + m - 1 of its subdomain: until
// the subdomain is at most `ahead` slices behind them.  One lane polls (the
// word's line is written at every step), the workgroup waits for it.  False when
// the subdomain is past them: a helper that is late goes on to the next chunk.
__device__ __forceinline__ bool helper_wait(const int *prog, int from, int i0, int m, int ahead) {
    __shared__ int at;
    if (threadIdx.x == 0) {
        int done = 0;
        for (int spin = 0; spin < PSPIN; spin++) {
            done = max(__hip_atomic_load(prog, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - from, -1);
            if (i0 - done <= ahead) break;
            __builtin_amdgcn_s_sleep(8);
        }
        at = done;
    }
    __syncthreads();
    bool take = at < i0 + m;
    __syncthreads();
    return take;
}

// Helper j of H of subdomain s: reads the data of the slices up to BPD ahead of
// the factorisation into the XCD's L2, in chunks of BPC.
constexpr int BPC = 8, BPD = 64, BHELP = 4;
__device__ unsigned bilu_prefetch(const FactArgs &A, int s, int j, int H) {
    const int s0 = A.soff[A.lbase[s]], nsl = A.soff[A.lbase[s] + A.nlev[s]] - s0;
    unsigned acc = 0;
    for (int c = j; c * BPC < nsl; c += H) {
        const int i0 = c * BPC;
        const long f = s0 + i0, m = min(BPC, nsl - i0);
        if (!helper_wait(&A.prog[PROG_STRIDE * s], 0, i0, (int)m, BPD)) continue;
        Lines<8> l;
        l.set(0, A.lval + 4 * f * RAS_MENT, 32L * RAS_MENT * m);
        l.set(1, A.tval + 4 * f * RAS_MENT, 32L * RAS_MENT * m);
        l.set(2, A.dinv + 4 * f * RAS_ROWS, 32L * RAS_ROWS * m);
        l.set(3, A.lcol + f * RAS_MENT, 4L * RAS_MENT * m);
        l.set(4, A.ldiag + f * RAS_MENT, 4L * RAS_MENT * m);
        l.set(5, A.glob + f * RAS_ROWS, 4L * RAS_ROWS * m);
        l.set(6, A.nl + f * RAS_ROWS, 4L * RAS_ROWS * m);
        l.set(7, A.xptr + f * RAS_ROWS, 4L * RAS_ROWS * m);
        acc += l.touch();
    }
    return acc;
}

__global__ __launch_bounds__(BWG) void k_bilu0(FactArgs A) {
    __shared__ int count;
    const int s = blockIdx.x % A.nsp, hj = (int)blockIdx.x / A.nsp - 1;
    if (s >= A.ns) return;
    if (hj >= 0) {
        // a helper, on its subdomain's XCD (see k_ras_sweep)
        unsigned acc = bilu_prefetch(A, s, hj, A.nhelp);
        if (A.nhelp < 0) A.prog[0] = (int)acc;     // never taken; keeps the reads
        return;
    }
    if (threadIdx.x == 0) count = 0;
    __syncthreads();
    const int nlev = A.nlev[s];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool h = lane & 1;
    // scalar loads: a vector load's wait would be for all before it as well
    const auto *soff = (const __attribute__((address_space(4))) int *)(A.soff + A.lbase[s]);
    const int s0 = soff[0], s1 = soff[nlev];
    int sl = s0 + wave, seen = 0;
    if (sl >= s1) return;
    // the level of slice sl: its first slice and the next level's
    int L = 0, lo = s0, hi = soff[1];
    auto level_of = [&](int t) {
        while (t >= hi) {
            L++;
            lo = hi;
            hi = soff[L + 1];
        }
    };
    level_of(sl);
    // one slice, R, while the wavefront's next one's data are requested into N
    auto slice = [&](BiluRow &R, BiluRow &N) __attribute__((always_inline)) {
        const int need = lo - s0;
        while (seen < need)
            seen = __builtin_amdgcn_readfirstlane(
                __hip_atomic_load(&count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        double dk[2][4];
#pragma unroll
        for (int i = 0; i < 2; i++) ld4(dk[i], &A.dinv[4 * (long)(R.q[i] >= 0 ? R.q[i] : R.p)]);
        // block rows h, 1 - h of the lane's second entry: the partner holds one
        double2 a2[2], u2[2];
        {
            double2 t = sel2(h, R.a1[0], R.a1[1]);
            a2[0] = sel2(h, R.a1[1], R.a1[0]);
            a2[1] = make_double2(dpp_move<DPP_XOR1>(t.x), dpp_move<DPP_XOR1>(t.y));
            t = sel2(h, R.u1[0], R.u1[1]);
            u2[0] = sel2(h, R.u1[1], R.u1[0]);
            u2[1] = make_double2(dpp_move<DPP_XOR1>(t.x), dpp_move<DPP_XOR1>(t.y));
        }
        // U_qp that extra matches change
#pragma unroll
        for (int i = 0; i < 2; i++)
            if (R.kd[i] >= 0) {
                const double2 *u = (const double2 *)A.uval;
                double2 x = u[ras_val(R.kd[i], h) >> 1], y = u[ras_val(R.kd[i], 1 - h) >> 1];
                if (i == 0) { R.u0[0] = x; R.u0[1] = y; }
                else { u2[0] = x; u2[1] = y; }
            }
        // (behind the wavefront's last slice: that one once more)
        const int nx = sl + BNW < s1 ? sl + BNW : sl;
        bilu_load(A, N, nx, lane);
        // entries of a row whose main entries are all (NOT_PLAIN if there are
        // more, or extra matches), -1 for no row
        constexpr int NOT_PLAIN = 2 * LPF + 1;
        const bool row = R.glob >= 0;
        const int info = !row ? -1 : (R.xi == R.xe ? min(R.nlp, NOT_PLAIN) : NOT_PLAIN);
        const bool plain = info < NOT_PLAIN;
        // the second position of a plain row, with its entries LPF ..
        const int info2 = dpp_move<DPP_XOR2>(info);
        const bool second = (lane & 2) && !row && info2 > LPF && info2 < NOT_PLAIN;
        const int nst = second ? info2 - LPF : (plain ? info : 0);
        // entry h (rows h, 1 - h), entry 2 + h
        double2 l0[2], l1[2], p0[2], p1[2];
        const double2 zero = make_double2(0.0, 0.0);
#pragma unroll
        for (int j = 0; j < 2; j++) {
            const double2 a = R.a0[j], b = a2[j];
            l0[j] = make_double2(a.x * dk[0][0] + a.y * dk[0][2], a.x * dk[0][1] + a.y * dk[0][3]);
            l1[j] = make_double2(b.x * dk[1][0] + b.y * dk[1][2], b.x * dk[1][1] + b.y * dk[1][3]);
            // subtracting zero changes nothing
            p0[j] = sel2(R.kd[0] != -1, row_prod(l0[j], R.u0[0], R.u0[1], h), zero);
            p1[j] = sel2(R.kd[1] != -1, row_prod(l1[j], u2[0], u2[1], h), zero);
        }
        auto other = [](double2 v) {
            return make_double2(dpp_move<DPP_XOR1>(v.x), dpp_move<DPP_XOR1>(v.y));
        };
        const double2 r0 = other(p0[1]), r1 = other(p1[1]), rl = other(l1[1]);
        double2 d = R.d;
        const double2 d0 = other(d);
        auto sub = [&](double2 v) { d.x -= v.x; d.y -= v.y; };
        const double2 w0 = sel2(h, r0, p0[0]), w1 = sel2(h, p0[0], r0);
        const double2 w2 = sel2(h, r1, p1[0]), w3 = sel2(h, p1[0], r1);
        sub(w0);
        sub(w1);
        sub(w2);
        sub(w3);
        const bool lng = plain && info > LPF;
        if (__ballot(lng)) {
            auto next = [&](double2 v) {
                double2 t = make_double2(dpp_move<DPP_XOR2>(v.x), dpp_move<DPP_XOR2>(v.y));
                sub(sel2(lng, t, zero));
            };
            next(w0);
            next(w1);
            next(w2);
            next(w3);
        }
        {
            double2 *lv = (double2 *)A.lval + 2 * (long)sl * RAS_MENT + lane;
            if ((int)h < nst) { lv[0] = l0[0]; lv[64] = l0[1]; }
            if (2 < nst) lv[128] = sel2(h, rl, l1[0]);
            if (3 < nst) lv[192] = sel2(h, l1[0], rl);
        }
        if (__ballot(row && !plain)) {
            double D[4] = {R.d.x, R.d.y, d0.x, d0.y};      // the first lane's view
            if (row && !plain && !h) {
                const RasRow rl(A.xlb, R.p), ru(A.xub, R.p);
                for (int e = 0; e < R.nlp; e++) {
                    long k = rl(e);
                    int qe = A.lcol[k], kde = A.ldiag[k];
                    double ae[4], dke[4], ude[4];
                    ld_blk(ae, A.lval, k);      // an earlier entry's extra match may have changed it
                    ld4(dke, &A.dinv[4 * (long)qe]);
                    if (kde == -2) ld_blk(ude, A.tval, k);
                    else if (kde >= 0) ld_blk(ude, A.uval, kde);
                    bilu_entry(A, rl, ru, R.nlp, e, ae, dke, kde, ude, D, R.xi, R.xe);
                }
            }
            const double2 D1 = other(make_double2(D[2], D[3]));
            if (!plain) d = h ? D1 : make_double2(D[0], D[1]);
        }
        const double2 o = other(d);
        const double t = d.x * o.y - d.y * o.x, det = h ? -t : t;
        if (row) {
            if (det == 0.0 || det != det) atomicOr(A.status, 1);
            const double2 z = make_double2(h ? -d.x : o.y, h ? o.x : -d.y);
            ((double2 *)A.dinv)[(long)sl * 64 + lane] = make_double2(z.x / det, z.y / det);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        // one lane adds (an atomicAdd here comes with instructions that combine lanes)
        if (lane == 0)
            asm volatile("ds_add_u32 %0, %1"
                         :: "v"((unsigned)(size_t)(__attribute__((address_space(3))) int *)&count), "v"(1)
                         : "memory");
        if (wave == 0)      // the slice it is at (see sweep_step)
            __hip_atomic_store(&A.prog[PROG_STRIDE * blockIdx.x], sl - s0, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
        level_of(nx);
        sl += BNW;
    };
    BiluRow X, Y;
    bilu_load(A, X, sl, lane);
    while (sl < s1) {
        slice(X, Y);
        if (sl < s1) slice(Y, X);
    }
}

template <class T>
__global__ void k_cast(long n, const double *a, T *b) {
    long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i < n) b[i] = (T)a[i];
}

// ------------------------------------------------------------------ solve
// Restriction of r to the overlapped subdomains, into local (level) order:
// one thread per local row in natural order, so that the reads of r are
// contiguous along the tiles' rows; each row's pair lands at its position.
template <class T>
__global__ void k_ras_gather(int mtot, const int *glob_nat, const int *pos, const double *r,
                             T *rl, int *prog, int ns) {
    int l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l < ns) prog[PROG_STRIDE * l] = 0;   // the sweeps' progress counters (read by the helpers)
    if (l >= mtot) return;
    long g = glob_nat[l], p = pos[l];
    const double2 v = ((const double2 *)r)[g];
    rl[2 * p] = (T)v.x;
    rl[2 * p + 1] = (T)v.y;
}

// Restricted scatter: owned rows only; optional Pi_p addend on the pressure
// and accumulation into out (out = (out + Pi_p xp) + z, Algorithm 2's order).
// One thread per local row in natural order, like the gather, so that the
// writes to out are contiguous along the tiles' rows; each row reads its pair
// at its position.
template <class T>
__global__ void k_ras_scatter(int mtot, int n, const int *glob_nat, const unsigned char *owned_nat,
                              const int *pos, const T *y, const double *xp, int accumulate,
                              double *out) {
    int l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= mtot || !owned_nat[l]) return;
    long g = glob_nat[l], p = pos[l];
    double o0 = (double)y[2 * p], o1 = (double)y[2 * p + 1];
    if (accumulate) {
        double v0 = out[2 * g];
        if (xp && g < n) v0 += xp[g];
        out[2 * g] = v0 + o0;
        out[2 * g + 1] += o1;
    } else {
        if (xp && g < n) o0 += xp[g];
        out[2 * g] = o0;
        out[2 * g + 1] = o1;
    }
}

template <class T>
struct SweepArgs {
    const int *lbase, *nlev, *soff;
    const int4 *mL, *mU;         // per slice (see k_sweep_cols)
    const int *lcol, *ucol;      // main entries: slice, lane, pair; overflow as in RasRow
    const T *lval, *uval, *dinv, *rl;
    const double *zeros;         // as many bytes as a slice's main entries take
    T *y;
    int *prog;                   // PROG_STRIDE ns: slice each sweep is at (forward, then backward),
                                 // one counter per 256 bytes
    int ns;                      // subdomains (sweep workgroups)
    int nsp, nhelp;              // ns to a multiple of 8; prefetch workgroups per subdomain: workgroup
                                 // nsp (1 + j) + s is helper j of subdomain s
    int ahead;                   // slices a helper reads ahead of its sweep
};

// LDS ring of the results of recently finished rows: position p sits in
// slot p mod RING.  While level L is being computed, a finished position q
// is still in the ring when no position written after it has the same slot.
// Positions written after q lie in q's own level (concurrently) or in later
// levels up to L, so with every level narrower than RING the test is
// forward q >= end(L) - RING, backward q < start(L) + RING; with a wider
// level the window is empty and such entries come from global memory.
constexpr int RING_BYTES = 128 * 1024;
template <class T>
struct RingSize {
    static constexpr int rows = RING_BYTES / (2 * (int)sizeof(T));
};

template <class T>
struct Vec2 {
    typedef T type __attribute__((ext_vector_type(2)));
};
// The data of one task (slice) held by lane 2r + h for position r: component h
// of the right-hand side and, backward, row h of the inverse diagonal block;
// the blocks of entry h (rows h, 1 - h) and rows h of those of entries 2 and 3
// (3: where a row of the slice has it); the y values of entries h and
// 2 + h.
template <class T>
struct Task {
    typedef typename Vec2<T>::type V2;
    T a;
    V2 d, keep, send, v2, v3;
    V2 y[MAXK];
};

// Slice of task j of a wavefront: the wavefronts take the slices of the
// subdomain in turn (forward from the first, backward from the last).  Past
// the wavefront's last task the last one is repeated (prefetches only).
template <bool FWD, int NCW>
__device__ __forceinline__ int task_slice(int sa, int sb, int wave, int j, int nt) {
    int jj = j < nt ? j : nt - 1;
    return FWD ? sa + wave + NCW * jj : sb - 1 - wave - NCW * jj;
}

// Loads at a wavefront-uniform address plus this lane's byte offset, kept in
// scalar registers and one vector register (the asm stops the compiler from
// adding them up outside the loop, which takes a vector add per load).
typedef const __attribute__((address_space(1))) char *LaneBase;
template <class V>
__device__ __forceinline__ V ld_lane(const void *base, unsigned off) {
    LaneBase p = (LaneBase)base;
    asm("" : "+s"(p), "+v"(off));
    return *(const __attribute__((address_space(1))) V *)(p + off);
}

template <class T, bool FWD>
__device__ __forceinline__ void load_cols(int (&c)[MAXK], const SweepArgs<T> &A, int sl, unsigned lane) {
    typedef int I2 __attribute__((ext_vector_type(2)));
    I2 v = ld_lane<I2>((FWD ? A.lcol : A.ucol) + (long)sl * RAS_MENT, lane * 8u);
    c[0] = v.x;
    c[1] = v.y;
}

// w: entries of the slice's longest row
template <class T, bool FWD>
__device__ __forceinline__ void load_task(Task<T> &R, const SweepArgs<T> &A, int sl, int w, unsigned lane) {
    typedef typename Vec2<T>::type V2;
    // position 32 sl + lane / 2, component lane & 1
    R.a = ld_lane<T>((FWD ? A.rl : A.y) + (long)sl * 2 * RAS_ROWS, lane * (unsigned)sizeof(T));
    if (!FWD) R.d = ld_lane<V2>(A.dinv + (long)sl * 4 * RAS_ROWS, lane * (unsigned)sizeof(V2));
    const LaneBase vals = (LaneBase)((FWD ? A.lval : A.uval) + (long)sl * (4 * RAS_MENT));
    // parts that no row of the slice has come from zeros that stay in cache: no
    // branch, so that the waits stay exact
    LaneBase v01 = w > 0 ? vals : (LaneBase)A.zeros, v23 = w > 2 ? vals : (LaneBase)A.zeros;
    unsigned off = lane * (unsigned)sizeof(V2);
    asm("" : "+s"(v01), "+s"(v23), "+v"(off));
    typedef const __attribute__((address_space(1))) V2 *G2;
    constexpr int part = 64 * (int)sizeof(V2);
    R.keep = *(G2)(v01 + off);
    R.send = *(G2)(v01 + off + part);
    R.v2 = *(G2)(v23 + off + 2 * part);
    if (w > 3) R.v3 = *(G2)(v23 + off + 3 * part);
}

// Zero for a column whose y value is loaded early.
__device__ __forceinline__ unsigned not_pre(int c) { return ((unsigned)c >> COL_BITS) ^ (unsigned)F_PRE; }

// Request the y values of the task's entries marked F_PRE: finished before the
// level the wavefront is at when it issues this load (two steps before the
// task) and outside the LDS ring's window of the task's level.  Few lanes have
// one, fewer two, and a load occupies the CU's load path for 16 cycles however
// few lanes take part: one load serves both entries, into y[0], and a lane's
// second takes another.
template <class T>
__device__ __forceinline__ void prefetch_y(Task<T> &R, const int (&c)[MAXK], const T *y) {
    typedef typename Vec2<T>::type V2;
    unsigned n0 = not_pre(c[0]), n1 = not_pre(c[1]);
    if (min(n0, n1) == 0) R.y[0] = *(const V2 *)&y[2 * (long)((n0 == 0 ? c[0] : c[1]) & COL_MASK)];
    if ((n0 | n1) == 0) R.y[1] = *(const V2 *)&y[2 * (long)(c[1] & COL_MASK)];
}

// The even or odd lane's value in both lanes of a pair.
constexpr int DPP_EVEN = 0xa0, DPP_ODD = 0xf5;
template <int CTRL, class V2>
__device__ __forceinline__ V2 dpp_move2(V2 v) {
    V2 r;
    r.x = dpp_move<CTRL>(v.x);
    r.y = dpp_move<CTRL>(v.y);
    return r;
}

// One step of a triangular sweep: task k of the wavefront (columns and
// metadata in buffers k mod 4, the rest in buffers k mod 2).  Once the count of
// finished slices covers every earlier level, task k's entries are read from
// the ring, its rows computed and stored to y and the ring, and the count
// raised.  Only then are task k+2's early y values and static data requested
// (into the buffers just used) and task k+4's columns and metadata: a CU takes
// 64 bytes of loads a cycle, so a slice's 5 KB hold up the instructions behind
// them for some 80 cycles, and behind the count they delay no other wavefront.
//
// What bounds a sweep: those loads (keep + send + v2, mostly not v3, columns,
// right-hand side, early y, result: about 0.2 ms per direction of 143,000
// positions on one CU) where levels are wide, else the chain count - ring -
// products - ring of a level, about 0.25 us.  An application at 2M cells, 16
// subdomains of 135,000 rows in 487 levels: 1,262 us with workgroup barriers
// between the levels, loads before the products and rows of more than four
// entries finished from memory; 883 with the count, loads after it and two
// positions for long rows; 817 with 16 wavefronts; 762 with the early y values
// of both entries in one load, no load for entry 3 where no row has one, and
// the addresses in scalar registers.
//
// LDS operations of a wavefront take effect in the order they are issued, so
// whoever reads the raised count finds the slice's results in the ring; the
// stores to y are issued before, and a CU's later loads find them.
template <class T, bool FWD, int U>
__device__ __forceinline__ void sweep_step(const SweepArgs<T> &A, T *ring, int *count, int sa, int sb,
                                           int wave, unsigned lane, int nt, int k, Task<T> (&B)[2],
                                           int (&C)[4][MAXK], int (&M)[4], int &seen) {
    typedef typename Vec2<T>::type V2;
    constexpr int R = RingSize<T>::rows;
    constexpr int NCW = Sweep<T>::ncw;
    Task<T> &cur = B[U & 1];
    const int need = __builtin_amdgcn_readlane(M[U], 0);
    const int w = __builtin_amdgcn_readlane(M[U], 1);
    const int xb = __builtin_amdgcn_readlane(M[U], 2);
    const int nlong = __builtin_amdgcn_readlane(M[U], 3);      // < 0: has F_SLOW entries
    // ready before the wait: which entries are in the ring and where, and the y
    // values loaded early
    unsigned long in0 = __ballot(not_pre(C[U][0]) != 0), in1 = __ballot(not_pre(C[U][1]) != 0);
    int s0 = (int)sizeof(V2) * (C[U][0] & (R - 1)), s1 = (int)sizeof(V2) * (C[U][1] & (R - 1));
    V2 &y0 = cur.y[0], &y1 = cur.y[1];
    if (not_pre(C[U][0]) != 0) y1 = y0;
    asm volatile("" : "+s"(in0), "+s"(in1), "+v"(s0), "+v"(s1), "+v"(y1.x), "+v"(y1.y) :: "memory");
    while (seen < need)
        seen = __builtin_amdgcn_readfirstlane(
            __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    asm volatile("" ::: "memory");
    if (__builtin_expect(__builtin_amdgcn_inverse_ballot_w64(in0), 1))
        y0 = *(const V2 *)((const char *)ring + s0);
    if (__builtin_expect(__builtin_amdgcn_inverse_ballot_w64(in1), 1))
        y1 = *(const V2 *)((const char *)ring + s1);
    if (nlong < 0) {
        if (((unsigned)C[U][0] >> COL_BITS) == (unsigned)F_SLOW)
            y0 = *(const V2 *)&A.y[2 * (long)(C[U][0] & COL_MASK)];
        if (((unsigned)C[U][1] >> COL_BITS) == (unsigned)F_SLOW)
            y1 = *(const V2 *)&A.y[2 * (long)(C[U][1] & COL_MASK)];
        __builtin_amdgcn_s_waitcnt(0);      // nothing of this rare path stays in flight
    }
    // component h of row r: te = (a if h = 0) - sum over even entries, to = (a if
    // h = 1) - sum over odd ones, each in order; unused entries hold a zero block
    // (their y, from the ring, is finite)
    const bool h = lane & 1;
    T nk = -cur.keep.x * y0.x - cur.keep.y * y0.y;
    T ns = -cur.send.x * y0.x - cur.send.y * y0.y;
    V2 ye = dpp_move2<DPP_EVEN>(y1);
    T x2 = cur.v2.x * ye.x + cur.v2.y * ye.y, x3 = 0;
    T nr = dpp_move<DPP_XOR1>(ns);
    T ak = cur.a + nk;
    T te = (h ? nr : ak) - x2, to = h ? ak : nr;
    if (w > 3) {
        V2 yo = dpp_move2<DPP_ODD>(y1);
        x3 = cur.v3.x * yo.x + cur.v3.y * yo.y;
        to -= x3;
    }
    const int ql = nlong & 63;
    if (ql && w > RAS_MAIN) {
        // the slice's first ql rows have their next entries in the next
        // position's lanes
        bool lg = (int)lane < 4 * ql;
        T kq = dpp_move<DPP_XOR2>(nk), rq = dpp_move<DPP_XOR2>(nr);
        T e2 = dpp_move<DPP_XOR2>(x2), e3 = dpp_move<DPP_XOR2>(x3);
        te += lg ? (h ? rq : kq) : (T)0;
        to += lg ? (h ? kq : rq) : (T)0;
        te -= lg ? e2 : (T)0;
        to -= lg ? e3 : (T)0;
    }
    if (w > 2 * RAS_MAIN) {
        // rows with more than 2 RAS_MAIN entries (well rows): the
        // rest from the overflow entries
        const int *cols = FWD ? A.lcol : A.ucol;
        const T *vals = FWD ? A.lval : A.uval;
        // in rounds of K slot pairs: a round's y values and blocks are requested
        // together with the next round's columns; pairs past the row's own
        // re-read its last and are masked.  One wavefront is at it, so what it
        // costs is its instructions: the addresses are a base for all lanes and
        // an offset per lane, made once (two by a block's parity, see ras_val).
        // A row of 700 entries: 56 us FP64, 36 FP32; 74 and 64 with 64-bit addresses
        // per lane, two pairs a round and its columns requested at its start.
        constexpr int K = LK<T>;
        static_assert(K % 2 == 0 && MAXK % 2 == 0, "pairs alternate between the parities");
        const int np = (w + 1) / 2, blk = xb >> 6;
        const unsigned sz = (unsigned)sizeof(T), hb = 128u * h;
        const bool odd = blk & 1;
        const unsigned e0 = 2 * lane * sz, e1 = (128 + 2 * lane) * sz, f0 = (hb + 2 * lane) * sz,
                       f1 = (hb + 2 * (lane ^ 1)) * sz;
        const unsigned o0[2] = {odd ? f0 : e0, odd ? e0 : f0}, o1[2] = {odd ? f1 : e1, odd ? e1 : f1};
        int q[K];
        auto columns = [&](int k0) {
#pragma unroll
            for (int j = 0; j < K; j++)
                q[j] = ld_lane<int>(cols + 64L * (blk + min(k0 + j, np - 1)), lane * 4u);
        };
        columns(2 * MAXK);
        for (int k0 = 2 * MAXK; k0 < np; k0 += K) {
            V2 gv[K], ov[K], b0[K], b1[K];
            bool ok[K], inwin[K];
#pragma unroll
            for (int j = 0; j < K; j++) {
                ok[j] = k0 + j < np && q[j] >= 0;
                inwin[j] = ((unsigned)q[j] >> COL_BITS) == (unsigned)F_RING;
                unsigned qs = q[j] >= 0 ? (unsigned)(q[j] & COL_MASK) : 0u;
                const T *v = vals + 256L * (blk + min(k0 + j, np - 1));
                gv[j] = ld_lane<V2>(A.y, qs * (unsigned)sizeof(V2));
                ov[j] = *(const V2 *)&ring[2 * (qs & (R - 1))];
                b0[j] = ld_lane<V2>(v, o0[j & 1]);
                b1[j] = ld_lane<V2>(v, o1[j & 1]);
            }
            columns(k0 + K);
#pragma unroll
            for (int j = 0; j < K; j++) {
                T a0 = inwin[j] ? ov[j].x : gv[j].x, a1 = inwin[j] ? ov[j].y : gv[j].y;
                T e0 = b0[j].x * a0 + b0[j].y * a1;
                T e1 = b1[j].x * a0 + b1[j].y * a1;
                e0 = ok[j] ? e0 : (T)0;
                e1 = dpp_move<DPP_XOR1>(ok[j] ? e1 : (T)0);
                te -= h ? e1 : e0;
                to -= h ? e0 : e1;
            }
        }
        __builtin_amdgcn_s_waitcnt(0);
    }
    T out = te + to;
    if (!FWD) out = cur.d.x * dpp_move<DPP_EVEN>(out) + cur.d.y * dpp_move<DPP_ODD>(out);
    const int sl = task_slice<FWD, NCW>(sa, sb, wave, k, nt);
    // positions without a row store too: nothing reads those
    *(T *)((char *)(A.y + (long)sl * 2 * RAS_ROWS) + lane * (unsigned)sizeof(T)) = out;
    ring[(sl * 2 * RAS_ROWS + lane) & (2 * R - 1)] = out;
    // one lane adds (an atomicAdd here comes with a dozen instructions that
    // combine lanes, between the results and the count)
    if (lane == 0)
        asm volatile("ds_add_u32 %0, %1"
                     :: "v"((unsigned)(size_t)(__attribute__((address_space(3))) int *)count), "v"(1)
                     : "memory");
    __builtin_amdgcn_sched_barrier(0);
    // marked entries of task k+2 (finished by now, outside its ring window)
    prefetch_y(cur, C[(U + 2) & 3], A.y);
    const int sl4 = task_slice<FWD, NCW>(sa, sb, wave, k + 4, nt);
    M[U] = ld_lane<int>((FWD ? A.mL : A.mU) + sl4, (lane & 3) * 4u);
    load_cols<T, FWD>(C[U], A, sl4, lane);
    load_task<T, FWD>(cur, A, task_slice<FWD, NCW>(sa, sb, wave, k + 2, nt),
                      __builtin_amdgcn_readlane(M[(U + 2) & 3], 1), lane);
    // a store the helpers poll: the slice this wavefront is at, which moves on
    // inside a level too and ends less than NCW slices before the last one, so
    // that no helper waits for a sweep that is over.  (The count a level waits
    // for stands still while a level runs: level 0 of a rough pressure field has
    // thousands of rows, and with it the helpers of its last slices ran into
    // their spin bound, over 14 ms a chunk.)  Workgroup scope is enough: it goes
    // through to the XCD's L2, where the helpers' polls read, and nothing of the
    // sweep's results depends on when they see it.
    if (wave == 0)
        __hip_atomic_store(&A.prog[PROG_STRIDE * blockIdx.x], (FWD ? 0 : sb - sa) + NCW * k,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __builtin_amdgcn_sched_barrier(0);
}

// One triangular sweep of a subdomain: forward (L, unit diagonal) or
// backward (U, then the inverse diagonal block).
template <class T, bool FWD>
__device__ __forceinline__ void sweep_dir(const SweepArgs<T> &A, T *ring, int *count,
                                          int sa, int sb, int wave, unsigned lane) {
    int nsl = sb - sa;
    constexpr int NCW = Sweep<T>::ncw;
    int nt = nsl > wave ? (nsl - wave + NCW - 1) / NCW : 0;
    if (nt <= 0) return;
    Task<T> B[2];
    int C[4][MAXK];
    int M[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        int sl = task_slice<FWD, NCW>(sa, sb, wave, j, nt);
        M[j] = ld_lane<int>((FWD ? A.mL : A.mU) + sl, (lane & 3) * 4u);
        load_cols<T, FWD>(C[j], A, sl, lane);
        if (j < 2) load_task<T, FWD>(B[j], A, sl, __builtin_amdgcn_readlane(M[j], 1), lane);
    }
    // enter the loop with nothing in flight, so that the wait counts the
    // compiler derives at its head follow the steady state
    __builtin_amdgcn_s_waitcnt(0);
    int seen = FWD ? 0 : nsl;
    for (int k = 0;; k += 4) {
        sweep_step<T, FWD, 0>(A, ring, count, sa, sb, wave, lane, nt, k, B, C, M, seen);
        if (k + 1 >= nt) break;
        sweep_step<T, FWD, 1>(A, ring, count, sa, sb, wave, lane, nt, k + 1, B, C, M, seen);
        if (k + 2 >= nt) break;
        sweep_step<T, FWD, 2>(A, ring, count, sa, sb, wave, lane, nt, k + 2, B, C, M, seen);
        if (k + 3 >= nt) break;
        sweep_step<T, FWD, 3>(A, ring, count, sa, sb, wave, lane, nt, k + 3, B, C, M, seen);
        if (k + 4 >= nt) break;
    }
}

// ------------------------------------------------------- prefetch helpers
template <class T>
constexpr int PCH = sizeof(T) == 4 ? 16 : 8;   // slices per helper chunk
constexpr int MAX_HELP = 8;       // helper workgroups per subdomain

// Helper j of subdomain s, one direction: chunks j, j + H, ... of PCH
// slices in the sweep's order; each waits (bounded) until the sweep is at
// most A.ahead slices behind it, then reads the chunk's metadata, columns,
// factor blocks and right-hand side (backward: the forward result and the
// inverse diagonal blocks), about 400 lines in one trip.
template <class T, bool FWD>
__device__ unsigned prefetch_dir(const SweepArgs<T> &A, int s, int j, int H, int sa, int sb) {
    const int4 *meta = FWD ? A.mL : A.mU;
    const int *cols = FWD ? A.lcol : A.ucol;
    const T *vals = FWD ? A.lval : A.uval;
    int nsl = sb - sa;
    unsigned acc = 0;
    for (int c = j; c * PCH<T> < nsl; c += H) {
        int i0 = c * PCH<T>, i1 = min(i0 + PCH<T>, nsl), m = i1 - i0;
        if (!helper_wait(&A.prog[PROG_STRIDE * s], FWD ? 0 : nsl, i0, m, A.ahead)) continue;
        long f = FWD ? sa + i0 : sb - i1;       // lowest slice of the chunk
        Lines<FWD ? 4 : 5> l;
        l.set(0, vals + 4 * f * RAS_MENT, 4L * (long)sizeof(T) * RAS_MENT * m);
        l.set(1, cols + f * RAS_MENT, 4L * RAS_MENT * m);
        l.set(2, (FWD ? A.rl : (const T *)A.y) + 2 * f * RAS_ROWS, 2L * (long)sizeof(T) * RAS_ROWS * m);
        l.set(3, meta + f, 16L * m);
        if constexpr (!FWD) l.set(4, A.dinv + 4 * f * RAS_ROWS, 4L * (long)sizeof(T) * RAS_ROWS * m);
        acc += l.touch();
    }
    return acc;
}

// Forward then backward substitution of one subdomain per workgroup on the
// gathered right-hand side; the result overwrites y in local order.
template <class T>
__global__ __launch_bounds__(Sweep<T>::wg) void k_ras_sweep(SweepArgs<T> A) {
    constexpr int R = RingSize<T>::rows;
    __shared__ __attribute__((aligned(16))) T ring[2 * R];
    __shared__ int count;            // finished slices, forward then backward
    const int s = blockIdx.x % A.nsp, hj = (int)blockIdx.x / A.nsp - 1;
    if (s >= A.ns) return;
    int nlev = A.nlev[s], base = A.lbase[s];
    int sa = A.soff[base], sb = A.soff[base + nlev];
    if (hj >= 0) {
        // a helper, on the same XCD as its subdomain's sweep (workgroup b goes
        // to XCD b mod 8, and nsp is a multiple of 8)
        unsigned acc = prefetch_dir<T, true>(A, s, hj, A.nhelp, sa, sb);
        acc += prefetch_dir<T, false>(A, s, hj, A.nhelp, sa, sb);
        if (A.nhelp < 0) A.prog[0] = (int)acc;     // never taken; keeps the reads
        return;
    }
    for (int i = threadIdx.x; i < 2 * R; i += Sweep<T>::wg) ring[i] = (T)0;
    if (threadIdx.x == 0) count = 0;
    __syncthreads();
    int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned lane = threadIdx.x & 63;
    sweep_dir<T, true>(A, ring, &count, sa, sb, wave, lane);
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_store(&A.prog[PROG_STRIDE * s], sb - sa, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
    sweep_dir<T, false>(A, ring, &count, sa, sb, wave, lane);
}

// Ring window of every subdomain: positions [end(L) - ring, end(L)) forward
// ([start(L), start(L) + ring) backward) are still in the LDS ring while
// level L runs when every level is narrower than the ring; else none is.
__global__ void k_sub_window(const int *lbase, const int *nlevs, const int *soff, int ring, int *win) {
    __shared__ int mw;
    int s = blockIdx.x, base = lbase[s], nlev = nlevs[s];
    if (threadIdx.x == 0) mw = 0;
    __syncthreads();
    int m = 0;
    for (int L = threadIdx.x; L < nlev; L += blockDim.x)
        m = max(m, RAS_ROWS * (soff[base + L + 1] - soff[base + L]));
    atomicMax(&mw, m);
    __syncthreads();
    if (threadIdx.x == 0) win[s] = mw <= ring ? ring : 0;
}

// The sweep's columns and metadata, one wavefront per slice: where the sweep
// finds each entry's y value follows from its fixed schedule (ncw wavefronts
// take a subdomain's slices in turn, forward from the first, backward from
// the last; the early loads of task j are issued at task j - 2 of the same
// wavefront, when every level before that task's has finished): in the ring
// window of the entry's level -> F_RING; else finished before that bound ->
// F_PRE; else F_SLOW.  The class goes into the column's top bits.  Metadata:
// the count of finished slices (forward, then backward) at which the slice may
// run, the entries of its longest row, its overflow start, and its long rows,
// with the sign bit set if it has F_SLOW entries.
template <bool FWD>
__global__ void k_sweep_cols(int ns, const int *lbase, const int *nlevs, const int *soff,
                             const int *win, const int *perm, const int *lev, const int *w,
                             const int *wlong, const int *xb, const int *cols, int ncw, int *out,
                             int4 *meta) {
    int sl = blockIdx.x, lane = threadIdx.x;
    int lo = 0, hi = ns - 1;                  // subdomain: the last one starting at or before sl
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (soff[lbase[mid]] <= sl) lo = mid; else hi = mid - 1;
    }
    int s = lo, base = lbase[s], nlev = nlevs[s];
    int sa = soff[base], sb = soff[base + nlev];
    // a slice's first position is always a row
    int L = lev[perm[RAS_ROWS * sl]], idx = FWD ? sl - sa : sb - 1 - sl;
    int bound;
    if (idx / ncw < 2) {
        bound = RAS_ROWS * (FWD ? sa : sb);      // nothing finished yet
    } else {
        int L2 = lev[perm[RAS_ROWS * (FWD ? sl - 2 * ncw : sl + 2 * ncw)]];
        bound = RAS_ROWS * soff[base + (FWD ? L2 : L2 + 1)];
    }
    int ws = win[s], lev0 = RAS_ROWS * soff[base + L], lev1 = RAS_ROWS * soff[base + L + 1];
    bool slow = false;
    auto mark = [&](int q, bool main) {
        if (q < 0) return q;
        bool inwin = FWD ? q >= lev1 - ws : q < lev0 + ws;
        bool pre = (FWD ? q < bound : q >= bound) && !inwin;
        slow |= main && !inwin && !pre;
        return q | ((inwin ? F_RING : (pre ? F_PRE : F_SLOW)) << COL_BITS);
    };
    long b = (long)sl * RAS_MENT;
    int2 c;
    c.x = mark(cols[b + lane], true);
    c.y = mark(cols[b + RAS_SLICE + lane], true);
    *(int2 *)&out[b + 2 * lane] = c;
    for (int k = 2 * MAXK; k < (w[sl] + 1) / 2; k++) {
        long e = (long)xb[sl] + (long)k * RAS_SLICE + lane;
        out[e] = mark(cols[e], false);
    }
    bool any = __any(slow);
    if (lane == 0) {
        int need = FWD ? soff[base + L] - sa : (sb - sa) + (sb - soff[base + L + 1]);
        meta[sl] = make_int4(need, w[sl], xb[sl], wlong[sl] | (any ? 1 << 31 : 0));
    }
}

// Prefetch workgroups per subdomain: as many as fit beside the sweeps, one
// workgroup per CU (a grid of whole rounds of 8 XCDs).  One alone does not keep
// up and delays the end: 128 subdomains at 2M cells 285 us with one each, 259
// with none; 64: 280 us with three each, 329 with none.
static int helpers(int ns, int most) {
    int h = std::min(most, 256 / ((ns + 7) / 8 * 8) - 1);
    return h > 1 ? h : 0;
}

// ----------------------------------------------------------------- set-up
int r2p_ras_setup(r2p_cpr *P, hipStream_t s) {
    double t0 = r2p_now_ms();
    R2P_TRY(r2p_ras_static(P, s));
    r2p_jacobian *J = P->J;
    r2p_model *m = J->m;
    const Phys &ph = m->ph;
    RasStatic &S = P->rs;
    RasDyn &D = P->rd;
    int mtot = S.mtot, ns = S.ns, order = P->o.order;
    R2P_TRY(D.lev.ensure(mtot));
    R2P_TRY(D.nlnat.ensure(mtot));
    R2P_TRY(D.nunat.ensure(mtot));
    R2P_TRY(D.pos.ensure(mtot));
    R2P_TRY(D.counters.ensure(64 + 2 * ns));
    R2P_TRY(D.prog.ensure(PROG_STRIDE * ns));
    R2P_TRY(P->pin.ensure(1 << 16));
    int nb = r2p_blocks(mtot, BS);
    // 1. levels of the dependency graph
    R2P_TRY(D.apred.ensure(S.nadj > 0 ? S.nadj : 1));
    R2P_TRY(D.succ4.ensure(mtot));
    k_pred_count<<<nb, BS, 0, s>>>(mtot, ph.n, order, J->phi_o.p, S.glob_nat.p, S.aptr.p, S.adj.p,
                                   D.apred.p, D.nlnat.p, D.nunat.p, D.succ4.p);
    R2P_LAUNCH();
    R2P_TRY(D.suboff.ensure(ns + 1));
    R2P_TRY(D.indeg.ensure(mtot));
    R2P_TRY(D.queue.ensure(mtot));
    R2P_HIP(hipMemcpyAsync(D.suboff.p, S.h_off.data(), sizeof(int) * (ns + 1), hipMemcpyHostToDevice, s));
    int *dnlev = D.counters.p + 64;
    int *hflag = (int *)P->pin.p;
    k_levels<<<ns, WG, 0, s>>>(D.suboff.p, S.aptr.p, S.adj.p, D.apred.p, D.succ4.p, D.nlnat.p,
                               D.indeg.p, D.queue.p, D.lev.p, dnlev);
    R2P_LAUNCH();
    // 2. level segments
    R2P_HIP(hipMemcpyAsync(hflag, dnlev, sizeof(int) * ns, hipMemcpyDeviceToHost, s));
    R2P_HIP(hipStreamSynchronize(s));
    D.h_nlev.assign(ns, 0);
    D.h_lbase.assign(ns + 1, 0);
    for (int t = 0; t < ns; t++) {
        D.h_nlev[t] = hflag[t];
        if (D.h_nlev[t] > MAXLEV) {
            r2p_set_error("subdomain %d has %d dependency levels (limit %d)", t, D.h_nlev[t], MAXLEV);
            return R2P_EINVAL;
        }
        D.h_lbase[t + 1] = D.h_lbase[t] + D.h_nlev[t];
    }
    int nseg = D.h_lbase[ns];
    D.nseg = nseg;
    R2P_TRY(D.lptr_dev.ensure(nseg + 1));
    R2P_TRY(D.nlong.ensure(nseg));
    R2P_TRY(D.soff.ensure(nseg + 1));
    R2P_TRY(D.sub_lbase.ensure(ns));
    R2P_TRY(D.sub_nlev.ensure(ns));
    R2P_HIP(hipMemcpyAsync(D.sub_lbase.p, D.h_lbase.data(), sizeof(int) * ns, hipMemcpyHostToDevice, s));
    R2P_HIP(hipMemcpyAsync(D.sub_nlev.p, D.h_nlev.data(), sizeof(int) * ns, hipMemcpyHostToDevice, s));
    R2P_HIP(hipMemsetAsync(D.lptr_dev.p, 0, sizeof(int) * (nseg + 1), s));
    R2P_HIP(hipMemsetAsync(D.nlong.p, 0, sizeof(int) * nseg, s));
    k_level_count<<<nb, BS, 0, s>>>(mtot, S.sub_of.p, D.lev.p, D.sub_lbase.p, D.nlnat.p, D.nunat.p,
                                    D.lptr_dev.p, D.nlong.p);
    R2P_LAUNCH();
    R2P_TRY(r2p_scan_int(D.lptr_dev.p, D.lptr_dev.p, nseg + 1, nullptr, P->iscratch, P->pin, s));
    // 3. slices of RAS_ROWS positions per level; positions: stable sort by
    // (level segment, long rows, descending predecessor count)
    k_slice_count<<<r2p_blocks(nseg + 1, BS), BS, 0, s>>>(nseg, D.lptr_dev.p, D.nlong.p, D.soff.p);
    R2P_LAUNCH();
    int nslice = 0;
    R2P_TRY(r2p_scan_int(D.soff.p, D.soff.p, nseg + 1, &nslice, P->iscratch, P->pin, s));
    if (nslice > (1 << COL_BITS) / RAS_ROWS) {
        r2p_set_error("%d local rows exceed the factor storage", mtot);
        return R2P_EINVAL;
    }
    int npos = RAS_ROWS * nslice;
    D.nslice = nslice;
    D.npos = npos;
    R2P_TRY(D.perm.ensure(npos));
    R2P_TRY(D.glob.ensure(npos));
    R2P_TRY(D.owned.ensure(npos));
    R2P_TRY(D.nl.ensure(npos));
    R2P_TRY(D.nu.ensure(npos));
    R2P_TRY(D.dsrc_pos.ensure(npos));
    R2P_HIP(hipMemsetAsync(D.perm.p, 0xff, sizeof(int) * (size_t)npos, s));
    R2P_HIP(hipMemsetAsync(D.glob.p, 0xff, sizeof(int) * (size_t)npos, s));
    R2P_HIP(hipMemsetAsync(D.owned.p, 0, (size_t)npos, s));
    R2P_HIP(hipMemsetAsync(D.nl.p, 0, sizeof(int) * (size_t)npos, s));
    R2P_HIP(hipMemsetAsync(D.nu.p, 0, sizeof(int) * (size_t)npos, s));
    {
        DBuf<unsigned> &key = P->ws.u[0], &val = P->ws.u[1], &kt = P->ws.u[2], &vt = P->ws.u[3];
        DBuf<int> &hist = P->ws.i[0];
        R2P_TRY(key.ensure(mtot));
        R2P_TRY(val.ensure(mtot));
        R2P_TRY(kt.ensure(mtot));
        R2P_TRY(vt.ensure(mtot));
        k_order_keys<<<nb, BS, 0, s>>>(mtot, S.sub_of.p, D.lev.p, D.sub_lbase.p, D.nlnat.p, D.nunat.p,
                                       key.p, val.p);
        R2P_LAUNCH();
        R2P_TRY(r2p_sort_pairs(key.p, val.p, kt.p, vt.p, mtot, r2p_bits_for(nseg) + 3, hist,
                               P->iscratch, P->pin, s));
        k_perm_gather<<<nb, BS, 0, s>>>(mtot, key.p, val.p, D.lptr_dev.p, D.nlong.p, D.soff.p,
                                        S.glob_nat.p, S.owned_nat.p, D.nlnat.p, D.nunat.p, S.dsrc.p, D.pos.p,
                                        D.perm.p, D.glob.p, D.owned.p, D.nl.p, D.nu.p, D.dsrc_pos.p);
        R2P_LAUNCH();
        R2P_HIP(hipStreamSynchronize(s));
    }
    double t1 = r2p_now_ms();
    P->ms_order = t1 - t0;       // membership (when rebuilt), levels and the local order
    // 4. entries: slice widths, overflow starts, columns and block sources
    int np = r2p_blocks(npos, BS);
    R2P_TRY(D.wl.ensure(nslice));
    R2P_TRY(D.wu.ensure(nslice));
    R2P_TRY(D.wlong.ensure(nslice));
    R2P_TRY(D.xl_b.ensure(nslice + 1));
    R2P_TRY(D.xu_b.ensure(nslice + 1));
    k_slice_width<<<np, BS, 0, s>>>(nslice, D.nl.p, D.nu.p, D.wl.p, D.wu.p, D.wlong.p, D.xl_b.p,
                                   D.xu_b.p);
    R2P_LAUNCH();
    int nlx = 0, nux = 0;
    R2P_TRY(r2p_scan_int(D.xl_b.p, D.xl_b.p, nslice + 1, &nlx, P->iscratch, P->pin, s));
    R2P_TRY(r2p_scan_int(D.xu_b.p, D.xu_b.p, nslice + 1, &nux, P->iscratch, P->pin, s));
    k_overflow_base<<<r2p_blocks(nslice, BS), BS, 0, s>>>(nslice, D.xl_b.p, D.xu_b.p);
    R2P_LAUNCH();
    const long nle = (long)nslice * RAS_MENT + nlx, nue = (long)nslice * RAS_MENT + nux;
    if (nle > 0x7fffffffL || nue > 0x7fffffffL) {
        r2p_set_error("%ld factor blocks exceed the factor storage", std::max(nle, nue));
        return R2P_EINVAL;
    }
    D.nlent = nle;
    D.nuent = nue;
    for (DBuf<int> *c : {&D.lcol, &D.lsw, &D.lsrc, &D.ldiag}) R2P_TRY(c->ensure(nle));
    for (DBuf<int> *c : {&D.ucol, &D.usw, &D.usrc}) R2P_TRY(c->ensure(nue));
    R2P_HIP(hipMemsetAsync(D.lcol.p, 0xff, sizeof(int) * (size_t)nle, s));
    R2P_HIP(hipMemsetAsync(D.ucol.p, 0xff, sizeof(int) * (size_t)nue, s));
    k_fill_entries<<<np, BS, 0, s>>>(npos, ph.n, order, J->phi_o.p, D.perm.p, S.glob_nat.p,
                                     S.aptr.p, S.adj.p, S.asrc.p, D.pos.p, D.glob.p, D.xl_b.p,
                                     D.xu_b.p, D.lcol.p, D.lsrc.p, D.ucol.p, D.usrc.p);
    R2P_LAUNCH();
    // 5. numeric factorisation in FP64
    R2P_TRY(D.f64.lval.ensure(4 * (size_t)nle));
    R2P_TRY(D.f64.uval.ensure(4 * (size_t)nue));
    R2P_TRY(D.f64.dinv.ensure(4 * (size_t)npos));
    // unused entries and positions stay zero (they are read)
    R2P_HIP(hipMemsetAsync(D.f64.lval.p, 0, sizeof(double) * 4 * (size_t)nle, s));
    R2P_HIP(hipMemsetAsync(D.f64.uval.p, 0, sizeof(double) * 4 * (size_t)nue, s));
    R2P_HIP(hipMemsetAsync(D.f64.dinv.p, 0, sizeof(double) * 4 * (size_t)npos, s));
    R2P_TRY(P->status.ensure(4));
    R2P_HIP(hipMemsetAsync(P->status.p, 0, sizeof(int), s));
    FactArgs F;
    F.B.vp = J->vp.p; F.B.vs = J->vs.p; F.B.cw = J->cw.p; F.B.wc = J->wc.p; F.B.wd = J->wd.p;
    F.B.nperf = ph.nperf;
    F.npos = npos;
    F.n = ph.n; F.nx = ph.nx; F.nxy = ph.nx * ph.ny;
    F.cell_perf = m->cell_perf.p;
    F.lbase = D.sub_lbase.p; F.nlev = D.sub_nlev.p; F.soff = D.soff.p;
    F.xlb = D.xl_b.p; F.xub = D.xu_b.p; F.glob = D.glob.p;
    F.nl = D.nl.p; F.nu = D.nu.p;
    F.dsrc = D.dsrc_pos.p; F.lsrc = D.lsrc.p; F.usrc = D.usrc.p;
    F.lcol = D.lcol.p; F.ucol = D.ucol.p;
    R2P_TRY(P->basis.ensure(4 * (size_t)nle));
    F.tval = P->basis.p;
    F.lval = D.f64.lval.p; F.uval = D.f64.uval.p; F.dinv = D.f64.dinv.p; F.status = P->status.p;
    R2P_TRY(D.xptr.ensure(npos + 1));
    R2P_HIP(hipMemsetAsync(D.ldiag.p, 0xff, sizeof(int) * (size_t)nle, s));
    R2P_HIP(hipMemsetAsync(D.xptr.p + npos, 0, sizeof(int), s));
    F.ldiag = D.ldiag.p; F.xptr = D.xptr.p; F.xl = nullptr;
    F.prog = D.prog.p; F.ns = ns; F.nsp = (ns + 7) / 8 * 8;
    F.nhelp = helpers(ns, BHELP);
    k_bilu_gather<<<np, BS, 0, s>>>(F);
    R2P_LAUNCH();
    // positions of wells and perforated cells (the level queue is free again)
    int *wlist = D.queue.p, *nwlist = D.counters.p;
    R2P_HIP(hipMemsetAsync(nwlist, 0, sizeof(int), s));
    k_bilu_sym<<<np, BS, 0, s>>>(F, wlist, nwlist);
    R2P_LAUNCH();
    k_bilu_sym_well<<<256, 256, 0, s>>>(F, wlist, nwlist, 0);
    R2P_LAUNCH();
    int nx = 0;
    R2P_TRY(r2p_scan_int(D.xptr.p, D.xptr.p, npos + 1, &nx, P->iscratch, P->pin, s));
    R2P_TRY(D.xl.ensure(nx));
    F.xl = D.xl.p;
    if (nx > 0) {
        k_bilu_sym_well<<<256, 256, 0, s>>>(F, wlist, nwlist, 1);
        R2P_LAUNCH();
    }
    k_bilu0<<<F.nhelp ? F.nsp * (1 + F.nhelp) : ns, BWG, 0, s>>>(F);
    R2P_LAUNCH();
    R2P_TRY(D.zeros.ensure(4 * RAS_MENT));
    R2P_HIP(hipMemsetAsync(D.zeros.p, 0, sizeof(double) * 4 * RAS_MENT, s));
    // the vectors' unused positions are read too: they start from zero
    const bool f32 = P->o.precision == R2P_FP32;
    if (f32) {
        R2P_TRY(D.f32.lval.ensure(4 * (size_t)nle));
        R2P_TRY(D.f32.uval.ensure(4 * (size_t)nue));
        R2P_TRY(D.f32.dinv.ensure(4 * (size_t)npos));
        k_cast<float><<<r2p_blocks(4L * nle, BS), BS, 0, s>>>(4L * nle, D.f64.lval.p, D.f32.lval.p);
        R2P_LAUNCH();
        k_cast<float><<<r2p_blocks(4L * nue, BS), BS, 0, s>>>(4L * nue, D.f64.uval.p, D.f32.uval.p);
        R2P_LAUNCH();
        k_cast<float><<<r2p_blocks(4L * npos, BS), BS, 0, s>>>(4L * npos, D.f64.dinv.p, D.f32.dinv.p);
        R2P_LAUNCH();
        R2P_TRY(P->t_rasf.ensure(2 * (size_t)npos));
        R2P_TRY(P->t_rlf.ensure(2 * (size_t)npos));
        R2P_HIP(hipMemsetAsync(P->t_rasf.p, 0, sizeof(float) * 2 * (size_t)npos, s));
        R2P_HIP(hipMemsetAsync(P->t_rlf.p, 0, sizeof(float) * 2 * (size_t)npos, s));
    } else {
        R2P_TRY(P->t_ras.ensure(2 * (size_t)npos));
        R2P_TRY(P->t_rl.ensure(2 * (size_t)npos));
        R2P_HIP(hipMemsetAsync(P->t_ras.p, 0, sizeof(double) * 2 * (size_t)npos, s));
        R2P_HIP(hipMemsetAsync(P->t_rl.p, 0, sizeof(double) * 2 * (size_t)npos, s));
    }
    // columns and metadata for the sweep of the precision set up
    {
        int ring = f32 ? RingSize<float>::rows : RingSize<double>::rows;
        int ncw = f32 ? Sweep<float>::ncw : Sweep<double>::ncw;
        R2P_TRY(D.swin.ensure(ns));
        R2P_TRY(D.meta_l.ensure(nslice));
        R2P_TRY(D.meta_u.ensure(nslice));
        k_sub_window<<<ns, 256, 0, s>>>(D.sub_lbase.p, D.sub_nlev.p, D.soff.p, ring, D.swin.p);
        R2P_LAUNCH();
        k_sweep_cols<true><<<nslice, 64, 0, s>>>(ns, D.sub_lbase.p, D.sub_nlev.p, D.soff.p, D.swin.p,
                                                 D.perm.p, D.lev.p, D.wl.p, D.wlong.p, D.xl_b.p, D.lcol.p, ncw,
                                                 D.lsw.p, D.meta_l.p);
        R2P_LAUNCH();
        k_sweep_cols<false><<<nslice, 64, 0, s>>>(ns, D.sub_lbase.p, D.sub_nlev.p, D.soff.p, D.swin.p,
                                                  D.perm.p, D.lev.p, D.wu.p, D.wlong.p, D.xu_b.p, D.ucol.p, ncw,
                                                  D.usw.p, D.meta_u.p);
        R2P_LAUNCH();
    }
    R2P_HIP(hipMemcpyAsync(hflag, P->status.p, sizeof(int), hipMemcpyDeviceToHost, s));
    R2P_HIP(hipStreamSynchronize(s));
    P->ms_ras = r2p_now_ms() - t1;
    if (*hflag) { r2p_set_error("singular diagonal block in block ILU(0)"); return R2P_ESINGULAR; }
    D.maxlev = 0;
    for (int t = 0; t < ns; t++) D.maxlev = std::max(D.maxlev, D.h_nlev[t]);
    return 0;
}

template <class T>
static int ras_solve_t(r2p_cpr *P, const double *r, double *out, const double *xp,
                       int accumulate, T *y, T *rl, const RasFactors<T> &F, hipStream_t s) {
    RasDyn &D = P->rd;
    int mtot = P->rs.mtot;
    int nb = r2p_blocks(mtot, BS);
    int ns = P->rs.ns;
    k_ras_gather<T><<<nb, BS, 0, s>>>(mtot, P->rs.glob_nat.p, D.pos.p, r, rl, D.prog.p, ns);
    R2P_LAUNCH();
    SweepArgs<T> A;
    A.lbase = D.sub_lbase.p; A.nlev = D.sub_nlev.p; A.soff = D.soff.p;
    A.mL = D.meta_l.p; A.mU = D.meta_u.p;
    A.lcol = D.lsw.p; A.ucol = D.usw.p;
    A.lval = F.lval.p; A.uval = F.uval.p; A.dinv = F.dinv.p; A.rl = rl; A.y = y;
    A.ns = ns; A.nsp = (ns + 7) / 8 * 8;
    A.prog = D.prog.p;
    A.nhelp = helpers(ns, MAX_HELP);
    // what the subdomains of an XCD have read ahead shares its 4 MB of L2: 128
    // slices are 0.8 MB in FP64, 256 in FP32.  FP32 with 128 instead of 256, 2M
    // cells: 64 subdomains 185 us instead of 196, 4 subdomains 1,511 instead of
    // 1,473 (FP64 with 64 instead of 128: 744 instead of 559 at 16)
    A.ahead = sizeof(T) == 4 && ns <= 16 ? 256 : 128;
    A.zeros = D.zeros.p;
    k_ras_sweep<T><<<A.nhelp ? A.nsp * (1 + A.nhelp) : ns, Sweep<T>::wg, 0, s>>>(A);
    R2P_LAUNCH();
    k_ras_scatter<T><<<nb, BS, 0, s>>>(mtot, P->J->m->ph.n, P->rs.glob_nat.p, P->rs.owned_nat.p,
                                       D.pos.p, y, xp,
                                       accumulate, out);
    R2P_LAUNCH();
    return 0;
}

int r2p_ras_solve(r2p_cpr *P, const double *r, double *out, const double *xp, int accumulate,
                  hipStream_t s) {
    if (P->o.precision == R2P_FP32)
        return ras_solve_t<float>(P, r, out, xp, accumulate, P->t_rasf.p, P->t_rlf.p, P->rd.f32, s);
    return ras_solve_t<double>(P, r, out, xp, accumulate, P->t_ras.p, P->t_rl.p, P->rd.f64, s);
}

// --------------------------------------------------------------- export
extern "C" int r2p_ras_info(r2p_cpr *P, int sub, int *nsub, int *m, int *nblk, int *nlevels) {
    if (!P || !P->ready) { r2p_set_error("CPR not set up"); return R2P_ESTATE; }
    if (nsub) *nsub = P->rs.ns;
    if (sub < 0 || sub >= P->rs.ns) return 0;
    int a = P->rs.h_off[sub], b = P->rs.h_off[sub + 1];
    if (m) *m = b - a;
    if (nlevels) *nlevels = P->rd.h_nlev[sub];
    if (nblk) {
        std::vector<int> nl(b - a), nu(b - a);
        R2P_HIP(hipMemcpy(nl.data(), P->rd.nlnat.p + a, sizeof(int) * (b - a), hipMemcpyDeviceToHost));
        R2P_HIP(hipMemcpy(nu.data(), P->rd.nunat.p + a, sizeof(int) * (b - a), hipMemcpyDeviceToHost));
        long t = 0;
        for (int i = 0; i < b - a; i++) t += nl[i] + nu[i];
        *nblk = (int)t;
    }
    return 0;
}

extern "C" int r2p_ras_export(r2p_cpr *P, int sub, int *glob, int *level, unsigned char *owned,
                              double *dinv, int *erow, int *ecol, double *eval, void *stream) {
    if (!P || !P->ready) { r2p_set_error("CPR not set up"); return R2P_ESTATE; }
    if (sub < 0 || sub >= P->rs.ns) { r2p_set_error("bad subdomain"); return R2P_EINVAL; }
    hipStream_t s = (hipStream_t)stream;
    R2P_HIP(hipStreamSynchronize(s));
    RasDyn &D = P->rd;
    const size_t npos = D.npos;
    auto pull = [&](const auto *src, size_t cnt, auto &dst) -> int {
        dst.resize(cnt);
        if (cnt) {
            hipError_t e = hipMemcpy(dst.data(), src, sizeof(dst[0]) * cnt, hipMemcpyDeviceToHost);
            if (e != hipSuccess) return r2p_hip_fail(e, "export", __FILE__, __LINE__);
        }
        return 0;
    };
    std::vector<int> g, pm, lv, nl, nu, so, xb[2], cc[2];
    std::vector<unsigned char> ow;
    std::vector<double> vv[2], dv;
    R2P_TRY(pull(D.glob.p, npos, g));
    R2P_TRY(pull(D.perm.p, npos, pm));
    R2P_TRY(pull(D.lev.p, (size_t)P->rs.mtot, lv));
    R2P_TRY(pull(D.nl.p, npos, nl));
    R2P_TRY(pull(D.nu.p, npos, nu));
    R2P_TRY(pull(D.soff.p, (size_t)D.nseg + 1, so));
    R2P_TRY(pull(D.xl_b.p, (size_t)D.nslice, xb[0]));
    R2P_TRY(pull(D.xu_b.p, (size_t)D.nslice, xb[1]));
    R2P_TRY(pull(D.lcol.p, (size_t)D.nlent, cc[0]));
    R2P_TRY(pull(D.ucol.p, (size_t)D.nuent, cc[1]));
    R2P_TRY(pull(D.f64.lval.p, 4 * (size_t)D.nlent, vv[0]));
    R2P_TRY(pull(D.f64.uval.p, 4 * (size_t)D.nuent, vv[1]));
    R2P_TRY(pull(D.f64.dinv.p, 4 * npos, dv));
    R2P_TRY(pull(D.owned.p, npos, ow));
    long k = 0, i = 0;
    int p0 = RAS_ROWS * so[D.h_lbase[sub]], p1 = RAS_ROWS * so[D.h_lbase[sub + 1]];
    // rows by level, descending predecessor count (up to 7), natural order
    std::vector<int> rows;
    for (int p = p0; p < p1; p++)
        if (pm[p] >= 0) rows.push_back(p);
    auto order = [&](int p) {
        return std::make_tuple(lv[pm[p]], 7 - std::min(nl[p], 7), pm[p]);
    };
    std::sort(rows.begin(), rows.end(), [&](int p, int q) { return order(p) < order(q); });
    for (int p : rows) {
        if (glob) glob[i] = g[p];
        if (level) level[i] = lv[pm[p]];
        if (owned) owned[i] = ow[p];
        if (dinv) memcpy(dinv + 4 * i, dv.data() + 4L * p, 4 * sizeof(double));
        i++;
        for (int part = 0; part < 2; part++) {
            const RasRow at(xb[part].data(), p);
            int cnt = part == 0 ? nl[p] : nu[p];
            for (int e = 0; e < cnt; e++, k++) {
                long idx = at(e);
                if (erow) erow[k] = g[p];
                if (ecol) ecol[k] = g[cc[part][idx]];
                if (eval)
                    for (int j = 0; j < 2; j++)
                        memcpy(eval + 4 * k + 2 * j, vv[part].data() + ras_val(idx, j),
                               2 * sizeof(double));
            }
        }
    }
    return 0;
}
