// Aggregation AMG on the pressure block A_pp (the M(A_pp)^-1 stage of the
// "Multi-stage preconditioner", Algorithm 2, with restriction Pi_r of Eq 34).
//
// The paper names AMG without fixing a variant.  Reading used here:
// strength -a_ij >= theta * max_{k!=i}(-a_ik) with -a_ij > 0; pairwise
// matching by handshakes (each unmatched row proposes its strongest
// unmatched strong neighbour, ties to the smaller index; mutual proposals
// pair up; `match_rounds` rounds); rows still unmatched join the pair of
// their strongest strong neighbour that is in a pair, else stay singletons;
// aggregates numbered by their leader (smaller row of the pair or the singleton); `agg_passes` passes per
// level, each on the Galerkin product of the previous one; piecewise-constant
// prolongation and Galerkin coarse matrices summed in ascending fine row and
// stored column order; l1-Jacobi smoothing (d_i = sum_j |a_ij|), one sweep
// before and after the coarse correction; V-cycle; the coarsest level is
// solved with its explicit inverse, computed once per set-up by dense LU
// with partial pivoting in FP64.
//
// Every set-up decision (strength, matching, joins, numbering) is integer
// work on values summed in a fixed order, so the hierarchy is reproducible.
// Compiled without floating-point contraction.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "r2p_impl.h"

constexpr int BS = 256;
constexpr int G = 4;                // lanes per row of the coarse-level row kernels
constexpr int KO_BLOCKS = 1024;     // grid of the K-cycle orthogonalisation pass

// ------------------------------------------------------- level 0 = A_pp
__global__ void k_app_count(Phys P, int *cnt) {
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= P.n) return;
    int nxy = P.nx * P.ny;
    int i = c % P.nx, j = (c / P.nx) % P.ny, k = c / nxy;
    cnt[c] = 1 + (i > 0) + (i + 1 < P.nx) + (j > 0) + (j + 1 < P.ny) + (k > 0) + (k + 1 < P.nz);
}

__global__ void k_app_cols(Phys P, const int *rp, int *col, int *slot) {
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= P.n) return;
    int nxy = P.nx * P.ny;
    int i = c % P.nx, j = (c / P.nx) % P.ny, k = c / nxy;
    int z = rp[c];
    const int order[7] = {5, 3, 1, 0, 2, 4, 6};
    bool ex[7] = {true, i > 0, i + 1 < P.nx, j > 0, j + 1 < P.ny, k > 0, k + 1 < P.nz};
    for (int oi = 0; oi < 7; oi++) {
        int sl = order[oi];
        if (!ex[sl]) continue;
        col[z] = c + slot_offset(sl, P.nx, nxy);
        slot[z] = sl;
        z++;
    }
}

__global__ void k_app_vals(int n, const int *rp, const int *slot, const double2 *vp, double *val) {
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    for (int z = rp[c]; z < rp[c + 1]; z++) val[z] = vp[(long)slot[z] * n + c].x;
}

// The same level-0 operator in the 7-slot stencil layout of the Jacobian
// (absent neighbours hold 0), for the coalesced level-0 cycle kernels.
__global__ void k_app_v7(int n, const double2 *vp, double *v7) {
    long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (t < 7L * n) v7[t] = vp[t].x;
}

// Rows of a CSR-like structure longer than a threshold: next-level rows with
// more than BIG members (restricted by a wavefront), and matrix rows with
// more than HEAVY entries (smoothed by a wavefront).  Aggregates that
// absorbed many unmatched rows make a few coarse rows hundreds of entries
// long; one thread per row would serialise the whole launch on them.
constexpr int BIG = 16;
constexpr int HEAVY = 32;
__global__ void k_long_flag(int n, const int *ptr, int thr, int *flag) {
    int I = blockIdx.x * blockDim.x + threadIdx.x;
    if (I < n) flag[I] = ptr[I + 1] - ptr[I] > thr;
    if (I == n) flag[I] = 0;
}

__global__ void k_long_list(int n, const int *ptr, int thr, const int *scan, int *list) {
    int I = blockIdx.x * blockDim.x + threadIdx.x;
    if (I < n && ptr[I + 1] - ptr[I] > thr) list[scan[I]] = I;
}

// ------------------------------------------------------------- matching
// The row scans below give a group of GS lanes to each row: lanes stride over
// the row's entries (ascending within a lane), then a butterfly combines the
// lanes.  The reductions are exact (a maximum, or the strongest column with
// ties to the smaller column, which is what a scan in ascending column order
// keeps), so the result equals the sequential one bit for bit.
constexpr int GS = 8;

__device__ __forceinline__ void row_group(int n, int &i, int &g) {
    i = blockIdx.x * (blockDim.x / GS) + (int)threadIdx.x / GS;
    g = threadIdx.x % GS;
    (void)n;
}

// (s, j) replaced by (s2, j2) when that is stronger, or as strong with a
// smaller column (j = -1: none).
__device__ __forceinline__ void take_stronger(double &s, int &j, double s2, int j2) {
    if (j2 >= 0 && (j < 0 || s2 > s || (s2 == s && j2 < j))) { s = s2; j = j2; }
}

// a_ji by binary search of row j (columns ascend), 0 when j stores no i.
__device__ __forceinline__ double entry_of(const int *rp, const int *col, const double *val, int j,
                                           int i) {
    int lo = rp[j], hi = rp[j + 1];
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        int c = col[mid];
        if (c == i) return val[mid];
        if (c < i) lo = mid + 1;
        else hi = mid;
    }
    return 0.0;
}

// Coupling weights w[z] = -(a_ij + a_ji)/2 of every stored off-diagonal
// entry z = (i, j) (0 on the diagonal), the same number from either row,
// and M_i = max(0, max_j w_ij).
__global__ void k_weights(int n, const int *rp, const int *col, const double *val, double *w,
                          double *M, int *match) {
    int i, g;
    row_group(n, i, g);
    if (i >= n) return;                        // whole groups leave together
    double mx = 0.0;
    for (int z = rp[i] + g; z < rp[i + 1]; z += GS) {
        int j = col[z];
        double wz = 0.0;
        if (j != i) wz = -(val[z] + entry_of(rp, col, val, j, i)) / 2.0;
        w[z] = wz;
        if (wz > mx) mx = wz;
    }
    mx = fmax(mx, dpp_move<DPP_XOR1>(mx));
    mx = fmax(mx, dpp_move<DPP_XOR2>(mx));
    mx = fmax(mx, dpp_move<DPP_HALF_MIRROR>(mx));
    if (g == 0) {
        M[i] = mx;
        match[i] = -1;
    }
}

// The symmetric strength relation: w_ij > 0 and w_ij reaches theta of the
// largest weight of row i or of row j.
__device__ __forceinline__ bool strong_pair(double wij, double Mi, double Mj, double theta) {
    return wij > 0.0 && (wij >= theta * Mi || wij >= theta * Mj);
}

// A matched row's M carries the sign bit (k_accept), so one gather tells both.
__device__ __forceinline__ bool matched(double M) { return __double2hiint(M) < 0; }

// Strongest strong neighbour j of an unmatched row i that is unmatched
// (propose) or matched (join), ties to the smaller column; -1 if none.  What
// bounds it: three loads that depend on one another, row - entry - M of its
// column (five, with a match array read before M: 2.9 ms in the 64 calls of a set-up
// of 2M cells, 1.8 so).
template <bool JOIN>
__device__ __forceinline__ void strongest(int n, const int *rp, const int *col, const double *w,
                                          const double *M, double theta, int *out) {
    int i, g;
    row_group(n, i, g);
    if (i >= n) return;
    double best = 0.0;
    int best_j = -1;
    const double Mi = M[i];
    const int z0 = rp[i], z1 = rp[i + 1];
    if (!matched(Mi)) {
        for (int z = z0 + g; z < z1; z += GS) {
            int j = col[z];
            double s = w[z], Mj = M[j];
            if (j == i || matched(Mj) != JOIN || !strong_pair(s, Mi, fabs(Mj), theta)) continue;
            if (s > best) { best = s; best_j = j; }
        }
    }
    take_stronger(best, best_j, dpp_move<DPP_XOR1>(best), dpp_move<DPP_XOR1>(best_j));
    take_stronger(best, best_j, dpp_move<DPP_XOR2>(best), dpp_move<DPP_XOR2>(best_j));
    take_stronger(best, best_j, dpp_move<DPP_HALF_MIRROR>(best), dpp_move<DPP_HALF_MIRROR>(best_j));
    if (g == 0) out[i] = best_j;
}

__global__ void k_propose(int n, const int *rp, const int *col, const double *w, const double *M,
                          double theta, int *prop) {
    strongest<false>(n, rp, col, w, M, theta, prop);
}

__global__ void k_accept(int n, const int *prop, int *match, double *M) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int j = prop[i];                           // -1 for a matched row
    if (j >= 0 && prop[j] == i) {
        match[i] = j;
        M[i] = -M[i];
    }
}

// Unmatched rows: strongest strong neighbour that is in a pair (or -1).
__global__ void k_join(int n, const int *rp, const int *col, const double *w, const double *M,
                       double theta, int *jt) {
    strongest<true>(n, rp, col, w, M, theta, jt);
}

__global__ void k_leader_flag(int n, const int *match, const int *jt, int *flag) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int j = match[i];
    flag[i] = (j >= 0 && i < j) || (j < 0 && jt[i] < 0);
}

__global__ void k_number(int n, const int *match, const int *jt, const int *cid, int *agg) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int j = match[i];
    int lead;
    if (j >= 0) lead = i < j ? i : j;
    else if (jt[i] < 0) lead = i;
    else {
        int k = jt[i];
        int mk = match[k];
        lead = k < mk ? k : mk;
    }
    agg[i] = cid[lead];
}

// Composition of a pass with the aggregation so far: agg[i] <- a[agg[i]].
__global__ void k_compose(int n, const int *a, int *agg) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) agg[i] = a[agg[i]];
}

__global__ void k_iota(int n, int *a) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = i;
}

// Member lists (CSR) of the aggregates, ascending within each list: every row
// takes a slot of its aggregate (in no fixed order), and its place in the list
// is then the number of smaller members.  Lists are a few rows long, so this
// costs a few reads per row where a sort by aggregate takes three passes.  The
// reads grow with the square of a list's length, and one matching round can
// leave a hub that thousands of rows join: a list of more than FEW members is
// reported in *hub (a pinned word, zeroed by the host) and left out, and the
// host has all lists sorted (k_member_keys).
constexpr int FEW = 1024;
__global__ void k_member_slot(int n, const int *agg, int *cnt, int *slot) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) slot[i] = atomicAdd(&cnt[agg[i]], 1);
}

__global__ void k_member_fill(int n, const int *agg, const int *mptr, const int *slot, int *list) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) list[mptr[agg[i]] + slot[i]] = i;
}

__global__ void k_member_order(int n, const int *agg, const int *mptr, const int *list, int *mem,
                               int *hub) {
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    int i = list[t], I = agg[i], a = mptr[I], b = mptr[I + 1], r = a;
    if (b - a > FEW) {
        if (t == a) *hub = 1;
        return;
    }
    for (int k = a; k < b; k++) r += list[k] < i;
    mem[r] = i;
}

__global__ void k_member_keys(int n, const int *agg, unsigned *key, unsigned *val) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) { key[i] = (unsigned)agg[i]; val[i] = (unsigned)i; }
}

// ------------------------------------------------------------- Galerkin
// A_c = P^T A P row by row: the stored entries a_ij of coarse row I's members
// (ascending fine row, then stored column) are the terms (agg(j), a_ij).  Equal
// columns are added in that order, and the sums stand in ascending column
// order.  A row's terms are compared with one another in LDS: the first of
// equal columns adds them up, its place is the number of smaller columns among
// the firsts.  Rows have 14 to 26 terms on average, and the pass reads and
// writes each term once; two stable radix sorts of all terms moved them a
// dozen times (13.9 million terms: 1.9 ms, 0.5 ms so).
//
// A group of GL lanes takes a coarse row of up to GL members and GE terms;
// longer ones go on a list and take a workgroup each (k_gal_long).  Comparing
// all terms of a row grows with their square: a product with a row of more than
// FEW terms, which takes very strong contrasts or one matching round, is
// reported in *hub, nothing of it is merged, and the host has all its terms
// sorted (k_gal_expand).  (One matching round at 2M cells leaves a row of 930,916
// terms.)
constexpr int GL = 16;
constexpr int GE = 64;
constexpr int NO_COL = 0x7fffffff;
struct GalArgs {
    int nc;
    const int *mptr, *mem, *rp, *col, *agg;
    const double *val;
    int *rpc;                    // counting: entries of every coarse row; then their starts
    int *colc;
    double *valc;
    int *list, *nlist;           // long rows; their number
    int *hub;                    // set if a row has more than FEW terms
};

// One of the group's terms per lane and slot, up to SL slots.
template <bool MERGE, int SL>
__device__ __forceinline__ void gal_row(const GalArgs &A, int I, int E, int nf, int l, int *key,
                                        const double *val) {
    int k[SL], rank[SL];
    double sum[SL];
    bool first[SL];
#pragma unroll
    for (int s = 0; s < SL; s++) {
        k[s] = key[l + GL * s];
        first[s] = l + GL * s < E;
        sum[s] = 0.0;
        rank[s] = 0;
    }
#pragma unroll 4
    for (int f = 0; f < nf; f++) {
        int kf = key[f];
        double vf = MERGE ? val[f] : 0.0;
#pragma unroll
        for (int s = 0; s < SL; s++) {
            bool eq = kf == k[s];
            first[s] &= !(eq & (f < l + GL * s));
            if (MERGE) sum[s] += eq ? vf : 0.0;
        }
    }
    if (!MERGE) {
        int cnt = 0;
#pragma unroll
        for (int s = 0; s < SL; s++)
            cnt += __popc((unsigned)(__ballot(first[s]) >> (threadIdx.x & 48)) & 0xffffu);
        if (l == 0 && E >= 0) A.rpc[I] = cnt;
        return;
    }
    // the group's lanes are in one wavefront, whose LDS operations keep order
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int s = 0; s < SL; s++) key[l + GL * s] = first[s] ? k[s] : NO_COL;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll 4
    for (int f = 0; f < nf; f++) {
        int kf = key[f];
#pragma unroll
        for (int s = 0; s < SL; s++) rank[s] += kf < k[s];
    }
    int base = E > 0 ? A.rpc[I] : 0;
#pragma unroll
    for (int s = 0; s < SL; s++)
        if (first[s]) {
            A.colc[base + rank[s]] = k[s];
            A.valc[base + rank[s]] = sum[s];
        }
}

template <bool MERGE>
__global__ __launch_bounds__(256) void k_gal_rows(GalArgs A) {
    __shared__ int key[256 / GL][GE], st[256 / GL][GL + 1], mz[256 / GL][GL];
    __shared__ double val[MERGE ? 256 / GL : 1][MERGE ? GE : 1];
    const int g = threadIdx.x / GL, l = threadIdx.x % GL;
    const int I = xcd_block(blockIdx.x, gridDim.x) * (256 / GL) + g;
    if (!MERGE && blockIdx.x == 0 && threadIdx.x == 0) A.rpc[A.nc] = 0;
    int a = I < A.nc ? A.mptr[I] : 0, m = I < A.nc ? A.mptr[I + 1] - a : 0;
    int z0 = 0, len = 0;
    if (m <= GL && l < m) {
        int i = A.mem[a + l];
        z0 = A.rp[i];
        len = A.rp[i + 1] - z0;
    }
    int inc = len;
    for (int d = 1; d < GL; d <<= 1) {
        int u = __shfl_up(inc, d, GL);
        if (l >= d) inc += u;
    }
    st[g][l + 1] = inc;
    if (l == 0) st[g][0] = 0;
    mz[g][l] = z0;
    int E = __shfl(inc, GL - 1, GL);          // -1: nothing to do here
    if (m > GL || E > GE) {
        if (!MERGE && l == 0) A.list[atomicAdd(&A.nlist[0], 1)] = I;
        E = -1;
    }
    if (I >= A.nc) E = -1;
    __syncthreads();
#pragma unroll
    for (int s = 0; s < GE / GL; s++) {
        int e = l + GL * s, k = 0;
        if (e < E) {
            while (e >= st[g][k + 1]) k++;
            int z = mz[g][k] + e - st[g][k];
            key[g][e] = A.agg[A.col[z]];
            if (MERGE) val[g][e] = A.val[z];
        } else {
            key[g][e] = NO_COL;
            if (MERGE) val[g][e] = 0.0;
        }
    }
    __syncthreads();
    int mx = max(E, __shfl_xor(E, 16, 64));
    mx = __builtin_amdgcn_readfirstlane(max(mx, __shfl_xor(mx, 32, 64)));
    const int nf = (mx + 3) & ~3;
    if (mx <= GL) gal_row<MERGE, 1>(A, I, E, nf, l, key[g], val[MERGE ? g : 0]);
    else if (mx <= 2 * GL) gal_row<MERGE, 2>(A, I, E, nf, l, key[g], val[MERGE ? g : 0]);
    else gal_row<MERGE, GE / GL>(A, I, E, nf, l, key[g], val[MERGE ? g : 0]);
}

// The rows on the list, a workgroup each: their terms, in LDS, compared with
// one another.  2M cells with a standard deviation of ln k of 2: up to 4,037
// such rows a pass and up to 909 terms a row (of 1: 2,653 and 566; of 4: 3,545
// and 1,670).
template <bool MERGE>
__global__ __launch_bounds__(256) void k_gal_long(GalArgs A) {
    __shared__ int key[FEW], fkey[MERGE ? FEW : 1], mem[3][256], part[4];
    __shared__ double val[MERGE ? FEW : 1];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nl = A.nlist[0];
    for (int q = blockIdx.x; q < nl; q += gridDim.x) {
        const int I = A.list[q], a = A.mptr[I], m = A.mptr[I + 1] - a;
        int E = FEW + 1;
        if (m <= FEW) {              // (a longer member list is not there)
            E = 0;
            for (int t = tid; t < m; t += 256) E += A.rp[A.mem[a + t] + 1] - A.rp[A.mem[a + t]];
            for (int d = 32; d > 0; d >>= 1) E += __shfl_xor(E, d, 64);
            if (lane == 0) part[wv] = E;
            __syncthreads();
            E = part[0] + part[1] + part[2] + part[3];
            __syncthreads();
        }
        if (E > FEW) {
            if (tid == 0) {
                *A.hub = 1;
                A.rpc[I] = 0;
            }
            continue;
        }
        // the terms, 256 members at a time: each member's first term, stored
        // entry and length, then 16 lanes copy a member's
        int off = 0;
        for (int t0 = 0; t0 < m; t0 += 256) {
            int t = t0 + tid, i = t < m ? A.mem[a + t] : 0;
            int z0 = A.rp[i], len = t < m ? A.rp[i + 1] - z0 : 0, inc = len;
            for (int d = 1; d < 64; d <<= 1) {
                int u = __shfl_up(inc, d, 64);
                if (lane >= d) inc += u;
            }
            if (lane == 63) part[wv] = inc;
            __syncthreads();
            int st = off + inc - len;
            for (int w = 0; w < 4; w++) {
                st += w < wv ? part[w] : 0;
                off += part[w];
            }
            mem[0][tid] = st;
            mem[1][tid] = z0;
            mem[2][tid] = len;
            __syncthreads();
            for (int r = tid / 16; r < min(m - t0, 256); r += 16)
                for (int k = tid % 16; k < mem[2][r]; k += 16) {
                    int z = mem[1][r] + k;
                    key[mem[0][r] + k] = A.agg[A.col[z]];
                    if (MERGE) val[mem[0][r] + k] = A.val[z];
                }
            __syncthreads();
        }
        int cnt = 0;
        for (int e = tid; e < E; e += 256) {
            const int k = key[e];
            unsigned first = 1;
#pragma unroll 8
            for (int f = 0; f < e; f++) first &= key[f] != k;
            cnt += first;
            if (MERGE) fkey[e] = first ? k : NO_COL;
        }
        if (!MERGE) {
            for (int d = 32; d > 0; d >>= 1) cnt += __shfl_xor(cnt, d, 64);
            if (lane == 0) part[wv] = cnt;
            __syncthreads();
            if (tid == 0) A.rpc[I] = part[0] + part[1] + part[2] + part[3];
            __syncthreads();
            continue;
        }
        __syncthreads();
        const int base = A.rpc[I];
        for (int e = tid; e < E; e += 256) {
            const int k = fkey[e];
            if (k == NO_COL) continue;
            int rank = 0;
            double sum = 0.0;
#pragma unroll 8
            for (int f = 0; f < E; f++) {
                rank += fkey[f] < k;
                sum += key[f] == k ? val[f] : 0.0;
            }
            A.colc[base + rank] = k;
            A.valc[base + rank] = sum;
        }
        __syncthreads();
    }
}

// The product by sorting all terms, stably by coarse column and then by coarse
// row: equal (I, J) terms stay in ascending (row, stored column) order, and are
// summed in that order.
__global__ void k_gal_expand(int n, const int *rp, const int *agg, unsigned *keyI, const int *col,
                             unsigned *keyJ, unsigned *idx) {
    int i, g;
    row_group(n, i, g);
    if (i >= n) return;
    unsigned I = (unsigned)agg[i];
    for (int z = rp[i] + g; z < rp[i + 1]; z += GS) {
        keyI[z] = I;
        keyJ[z] = (unsigned)agg[col[z]];
        idx[z] = (unsigned)z;
    }
}

__global__ void k_gather_u(int m, const unsigned *idx, const unsigned *src, unsigned *dst) {
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < m) dst[k] = src[idx[k]];
}

// keyI, keyJ: the terms' coarse rows and columns in sorted order.
__device__ __forceinline__ bool first_of_run(int k, const unsigned *keyI, const unsigned *keyJ) {
    return k == 0 || keyI[k] != keyI[k - 1] || keyJ[k] != keyJ[k - 1];
}
__global__ void k_gal_flags(int m, const unsigned *keyI, const unsigned *keyJ, int *flag) {
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < m) flag[k] = first_of_run(k, keyI, keyJ);
}

// The first term of every run of equal (I, J) records where its run starts;
// the run of output entry u is then [start[u], start[u + 1]).
__global__ void k_gal_runs(int m, int nc, const unsigned *keyI, const unsigned *keyJ,
                           const int *uidx, int *start, int *rpc, int nnzc) {
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k == 0) { rpc[nc] = nnzc; start[nnzc] = m; }
    if (k >= m || !first_of_run(k, keyI, keyJ)) return;
    start[uidx[k]] = k;
    if (k == 0 || keyI[k - 1] != keyI[k]) rpc[keyI[k]] = uidx[k];
}

// One thread per coarse entry, four terms' loads in flight at a time.
__global__ void k_gal_sum(int nnzc, const int *start, const unsigned *idx, const unsigned *keyJ,
                          const double *val, int *colc, double *valc) {
    int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= nnzc) return;
    int a = start[u], b = start[u + 1];
    double s = 0.0;
    int t = a;
    for (; t + 4 <= b; t += 4) {
        unsigned i0 = idx[t], i1 = idx[t + 1], i2 = idx[t + 2], i3 = idx[t + 3];
        double v0 = val[i0], v1 = val[i1], v2 = val[i2], v3 = val[i3];
        s += v0;
        s += v1;
        s += v2;
        s += v3;
    }
    for (; t < b; t++) s += val[idx[t]];
    colc[u] = (int)keyJ[a];
    valc[u] = s;
}

__global__ void k_l1(int n, const int *rp, const double *val, double *l1) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double s = 0.0;
    for (int z = rp[i]; z < rp[i + 1]; z++) s += fabs(val[z]);
    l1[i] = s;
}

template <class T>
__global__ void k_castv(long n, const double *a, T *b) {
    long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i < n) b[i] = (T)a[i];
}

// ------------------------------------------------------------- coarsest
// One workgroup per row of the dense matrix.
__global__ void k_to_dense(int n, const int *rp, const int *col, const double *val, double *a,
                           int *pos, int *chosen) {
    int i = blockIdx.x;
    double *row = a + (long)i * n;
    for (int j = threadIdx.x; j < n; j += blockDim.x) row[j] = 0.0;
    if (threadIdx.x == 0) pos[i] = chosen[i] = i;
    __syncthreads();
    // a row's columns are distinct
    for (int z = rp[i] + (int)threadIdx.x; z < rp[i + 1]; z += blockDim.x) row[col[z]] = val[z];
}

// LU with partial pivoting (largest magnitude, ties to the smaller position)
// in panels of NB columns: k_lu_panel (one workgroup) factorises the panel,
// k_lu_update (many workgroups) applies it to the columns right of it.  Rows
// never move: pos[r] is the position a row has or is at present, row[k] the
// row chosen at position k.  L stays in the rows of `a`; every pivot row's U
// part goes to u[k].  Each entry receives its updates one pivot at a time in
// ascending order, as the unblocked algorithm does, so the factors are the
// same.
// What bounds it: a chain of n pivot steps.  One workgroup doing the whole
// matrix read it from L2 at every step (about 400 rows: 6.8 ms); with the
// panel in registers a step is one reduction, two barriers and at most NB
// multiply-subtracts, and the rest of the matrix is updated once per panel by
// the whole chip (the same matrix: 13 panels of 41 us, 12 updates of 14 us).
// The state of a panel workgroup: RPT rows per thread, their panel columns
// from the current pivot's on in registers (column kk of the panel is r[q][0]
// when its turn comes), and the rows' positions.
template <int T, int RPT, int NB>
struct LuPanel {
    double r[RPT][NB];
    int ps[RPT];
    double (*sv)[T / 64], (*prow)[NB];
    int (*si)[T / 64];
};

// take() for the candidates of lanes i and i ^ D (one of them the lane's own),
// D 16 or 32.
template <int D, class F>
__device__ __forceinline__ void take_swapped(double v, int i, const F &take) {
    int2 t = __builtin_bit_cast(int2, v), a, b;
    int ia, ib;
    if (D == 16) { rows_swap16(t.x, a.x, b.x); rows_swap16(t.y, a.y, b.y); rows_swap16(i, ia, ib); }
    else { rows_swap32(t.x, a.x, b.x); rows_swap32(t.y, a.y, b.y); rows_swap32(i, ia, ib); }
    take(__builtin_bit_cast(double, a), ia);
    take(__builtin_bit_cast(double, b), ib);
}

// Pivots kk .. kk + 7 (below nb) with at most W panel columns left; false
// when a pivot is zero or not a number (the same in every thread).
template <int T, int RPT, int NB, int W>
__device__ __forceinline__ bool lu_steps(LuPanel<T, RPT, NB> &S, int n, int k0, int kk, int nb,
                                         double *a, double *u, int *row) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int end = min(kk + 8, nb);
    for (; kk < end; kk++) {
        const int k = k0 + kk, buf = kk & 1;
        double best = -1.0;
        int bi = n;
        // selects, not branches: this is the step's chain
        auto take = [&](double v, int i) {
            bool t = (v > best) | ((v == best) & (i < bi));
            best = t ? v : best;
            bi = t ? i : bi;
        };
#pragma unroll
        for (int q = 0; q < RPT; q++) take(S.ps[q] >= k ? fabs(S.r[q][0]) : -1.0, S.ps[q]);
        take(dpp_move<DPP_XOR1>(best), dpp_move<DPP_XOR1>(bi));
        take(dpp_move<DPP_XOR2>(best), dpp_move<DPP_XOR2>(bi));
        take(dpp_move<DPP_HALF_MIRROR>(best), dpp_move<DPP_HALF_MIRROR>(bi));
        take(dpp_move<DPP_ROR8>(best), dpp_move<DPP_ROR8>(bi));
        take_swapped<16>(best, bi, take);
        take_swapped<32>(best, bi, take);
        if (lane == 0) { S.sv[buf][wid] = best; S.si[buf][wid] = bi; }
        __syncthreads();
        best = S.sv[buf][lane & (T / 64 - 1)];
        bi = S.si[buf][lane & (T / 64 - 1)];
        take(dpp_move<DPP_XOR1>(best), dpp_move<DPP_XOR1>(bi));
        take(dpp_move<DPP_XOR2>(best), dpp_move<DPP_XOR2>(bi));
        if (T >= 512) take(dpp_move<DPP_HALF_MIRROR>(best), dpp_move<DPP_HALF_MIRROR>(bi));
        if (T >= 1024) take(dpp_move<DPP_ROR8>(best), dpp_move<DPP_ROR8>(bi));
        if (!(best > 0.0)) return false;
#pragma unroll
        for (int q = 0; q < RPT; q++) {
            if (S.ps[q] == bi) {
#pragma unroll
                for (int j = 0; j < W; j++) S.prow[buf][j] = S.r[q][j];
                row[k] = (int)threadIdx.x + q * T;
            }
            S.ps[q] = S.ps[q] == bi ? k : (S.ps[q] == k ? bi : S.ps[q]);
        }
        __syncthreads();
        if ((int)threadIdx.x < min(W, nb - kk))
            u[(long)k * n + k + threadIdx.x] = S.prow[buf][threadIdx.x];
        double inv = 1.0 / S.prow[buf][0];
#pragma unroll
        for (int q = 0; q < RPT; q++) {
            if (S.ps[q] > k) {
                double l = S.r[q][0] * inv;
                a[(long)((int)threadIdx.x + q * T) * n + k] = l;
#pragma unroll
                for (int j = 1; j < W; j++) S.r[q][j - 1] = S.r[q][j] - l * S.prow[buf][j];
            }
        }
    }
    if constexpr (W > 8) {
        if (kk < nb) return lu_steps<T, RPT, NB, W - 8>(S, n, k0, kk, nb, a, u, row);
    }
    return true;
}

template <int T, int RPT, int NB>
__global__ __launch_bounds__(T) void k_lu_panel(int n, int k0, double *a, double *u, int *pos,
                                                int *row, int *status) {
    __shared__ double sv[2][T / 64], prow[2][NB];
    __shared__ int si[2][T / 64];
    if (*status) return;
    const int nb = min(NB, n - k0);
    LuPanel<T, RPT, NB> S;
    S.sv = sv;
    S.prow = prow;
    S.si = si;
#pragma unroll
    for (int q = 0; q < RPT; q++) {
        int i = (int)threadIdx.x + q * T;
        S.ps[q] = i < n ? pos[i] : -1;
#pragma unroll
        for (int j = 0; j < NB; j++)
            S.r[q][j] = a[(long)min(i, n - 1) * n + k0 + min(j, nb - 1)];
#pragma unroll
        for (int j = 0; j < NB; j++) S.r[q][j] = j < nb ? S.r[q][j] : 0.0;
    }
    if (!lu_steps<T, RPT, NB, NB>(S, n, k0, 0, nb, a, u, row)) {
        if (threadIdx.x == 0) *status = 1;
        return;
    }
#pragma unroll
    for (int q = 0; q < RPT; q++)
        if (S.ps[q] >= k0) pos[(int)threadIdx.x + q * T] = S.ps[q];
}

// The columns right of a panel: a workgroup takes 64 columns and LU_R rows.
// Every wavefront solves the columns of U (unit lower triangle of the panel), a
// column to a lane and all of it in registers (written to u by the first row
// of workgroups), then subtracts the panel's multiples from its rows that are
// still active.  About 400 rows: 22.5 us with U in LDS and each wavefront on 16
// of the columns, 14.4 us so.
constexpr int LU_R = 32;
template <int NB>
__global__ __launch_bounds__(256, 2) void k_lu_update(int n, int k0, double *a, double *u,
                                                      const int *pos, const int *row,
                                                      const int *status) {
    __shared__ double lt[NB][NB], ls[LU_R][NB];
    if (*status) return;
    const int cx = threadIdx.x & 63, ty = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j0 = k0 + NB + blockIdx.x * 64, j = j0 + cx, i0 = blockIdx.y * LU_R;
    const int jj = min(j, n - 1);
    // lt[k][i]: multiplier of panel row i for pivot k
    for (int e = threadIdx.x; e < NB * NB; e += 256)
        lt[e % NB][e / NB] = a[(long)row[k0 + e / NB] * n + k0 + e % NB];
    for (int e = threadIdx.x; e < LU_R * NB; e += 256) {
        int i = i0 + e / NB;
        ls[e / NB][e % NB] = i < n ? a[(long)i * n + k0 + e % NB] : 0.0;
    }
    double uk[NB], t[LU_R / 4];
    bool act[LU_R / 4];
#pragma unroll
    for (int k = 0; k < NB; k++) uk[k] = a[(long)row[k0 + k] * n + jj];
#pragma unroll
    for (int q = 0; q < LU_R / 4; q++) {
        int i = i0 + 4 * q + ty;
        act[q] = i < n && pos[min(i, n - 1)] >= k0 + NB;
        t[q] = a[(long)min(i, n - 1) * n + jj];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NB; k++)
#pragma unroll
        for (int i = k + 1; i < NB; i++) uk[i] -= lt[k][i] * uk[k];
    if (j >= n) return;
    if (blockIdx.y == 0) {
#pragma unroll
        for (int k = 0; k < NB; k++)
            if (k % 4 == ty) u[(long)(k0 + k) * n + j] = uk[k];
    }
#pragma unroll
    for (int q = 0; q < LU_R / 4; q++) {
        if (!act[q]) continue;
#pragma unroll
        for (int k = 0; k < NB; k++) t[q] -= ls[4 * q + ty][k] * uk[k];
        a[(long)(i0 + 4 * q + ty) * n + j] = t[q];
    }
}

// L below U in position order: u[k][j] = a[row[k]][j], j < k.
__global__ void k_lu_gather(int n, const double *a, const int *row, const int *status, double *u) {
    if (*status) return;             // singular: no row was chosen from the failed pivot on
    int k = blockIdx.x;
    const double *src = a + (long)row[k] * n;
    for (int j = threadIdx.x; j < k; j += blockDim.x) u[(long)k * n + j] = src[j];
}

// Column c of the inverse from the LU factors f (position order), one
// wavefront per column: x = P e_c, then the unit-lower and upper triangular
// solves, each row's inner product split over the lanes (lane l holds x_l,
// x_l+64, .. in registers) and summed by a fixed butterfly.  The rows are
// taken in blocks of 64, so that the registers a row needs are fixed, and
// requested AH rows before they are used.  What bounds it is the chain of
// 2 n rows: a step is one row's products, one butterfly and one update (about
// 400 rows: 0.20 ms; 1.0 ms with each row requested at its use and the
// iterate in LDS, 0.28 ms with every register masked at every step, 0.39 ms
// with two columns per wavefront).  Written column-major,
// invT[c*n + i] = (A^-1)_ic, so the coarse solve reads it coalesced.
template <int NR, int AH>
__global__ __launch_bounds__(64) void k_dense_inv_col(int n, const double *f, const int *pos,
                                                      const int *status, double *invT) {
    if (*status) return;             // singular: the factors are incomplete
    const int c = blockIdx.x, lane = threadIdx.x;
    const int p = pos[c];
    // x: right-hand side and forward solution; z: the solution, zero until
    // known, so that neither inner product needs a mask
    double x[NR], z[NR], w[AH][NR];
#pragma unroll
    for (int t = 0; t < NR; t++) {
        x[t] = lane + 64 * t == p ? 1.0 : 0.0;
        z[t] = 0.0;
    }
    // registers t0 .. t1 of row i of the factors (past the matrix: an end row)
    auto fetch = [&](double (&b)[NR], int i, int t0, int t1) {
        const double *r = f + (long)min(max(i, 0), n - 1) * n;
#pragma unroll
        for (int t = 0; t < NR; t++)
            if (t >= t0 && t <= t1) b[t] = r[min(lane + 64 * t, n - 1)];
    };
    // forward: rows up to p would only add products with zeros
#pragma unroll
    for (int tb = 0; tb < NR; tb++) {
        const int i1 = min(64 * tb + 64, n);
        int i = max(64 * tb, p + 1);
        if (i >= i1) continue;
#pragma unroll
        for (int q = 0; q < AH; q++) fetch(w[q], i + q, 0, tb);
        for (; i < i1; i += AH) {
#pragma unroll
            for (int q = 0; q < AH; q++) {
                if (i + q < i1) {
                    double s = 0.0;
#pragma unroll
                    for (int t = 0; t < NR; t++)
                        if (t <= tb) s += w[q][t] * (t < tb || lane + 64 * t < i + q ? x[t] : 0.0);
                    s = wave_sum_down(s);
                    fetch(w[q], i + q + AH, 0, tb);
                    x[tb] = lane + 64 * tb == i + q ? x[tb] - s : x[tb];
                }
            }
        }
    }
#pragma unroll
    for (int tb = NR - 1; tb >= 0; tb--) {
        const int i1 = 64 * tb;
        int i = min(64 * tb + 63, n - 1);
        if (i < i1) continue;
#pragma unroll
        for (int q = 0; q < AH; q++) fetch(w[q], i - q, tb, NR - 1);
        for (; i >= i1; i -= AH) {
#pragma unroll
            for (int q = 0; q < AH; q++) {
                if (i - q >= i1) {
                    double s = 0.0;
#pragma unroll
                    for (int t = 0; t < NR; t++)
                        if (t >= tb) s += w[q][t] * z[t];
                    s = wave_sum_down(s);
                    double v = (x[tb] - s) / w[q][tb];
                    z[tb] = lane + 64 * tb == i - q ? v : z[tb];
                    fetch(w[q], i - q - AH, tb, NR - 1);
                }
            }
        }
    }
#pragma unroll
    for (int t = 0; t < NR; t++)
        if (lane + 64 * t < n) invT[(long)c * n + lane + 64 * t] = z[t];
}

// The same with the iterate in LDS, for matrices whose rows do not fit the
// registers (above 1,024 rows: an explicit max_coarse, or a stalled
// coarsening).
__global__ __launch_bounds__(64) void k_dense_inv_col_lds(int n, const double *f, const int *pos,
                                                          const int *status, double *invT) {
    extern __shared__ double xs[];
    if (*status) return;
    int c = blockIdx.x, lane = threadIdx.x, p = pos[c];
    for (int i = lane; i < n; i += 64) xs[i] = i == p ? 1.0 : 0.0;
    __syncthreads();
    for (int i = p + 1; i < n; i++) {
        double s = 0.0;
        for (int j = lane; j < i; j += 64) s += f[(long)i * n + j] * xs[j];
        s = wave_sum_down(s);
        __syncthreads();
        if (lane == 0) xs[i] -= s;
        __syncthreads();
    }
    for (int i = n - 1; i >= 0; i--) {
        double s = 0.0;
        for (int j = i + 1 + lane; j < n; j += 64) s += f[(long)i * n + j] * xs[j];
        s = wave_sum_down(s);
        __syncthreads();
        if (lane == 0) xs[i] = (xs[i] - s) / f[(long)i * n + i];
        __syncthreads();
    }
    for (int i = lane; i < n; i += 64) invT[(long)c * n + i] = xs[i];
}

// The inverse of the coarsest matrix (n <= 4096 rows) into P->cinv.
template <int T, int RPT, int NB>
static int dense_lu(r2p_cpr *P, int n, hipStream_t s) {
    for (int k0 = 0; k0 < n; k0 += NB) {
        k_lu_panel<T, RPT, NB><<<1, T, 0, s>>>(n, k0, P->lu.p, P->luu.p, P->lupos.p, P->lurow.p,
                                               P->astatus.p);
        R2P_LAUNCH();
        int rest = n - k0 - NB;
        if (rest <= 0) break;
        k_lu_update<NB><<<dim3(r2p_blocks(rest, 64), r2p_blocks(n, LU_R)), 256, 0, s>>>(
            n, k0, P->lu.p, P->luu.p, P->lupos.p, P->lurow.p, P->astatus.p);
        R2P_LAUNCH();
    }
    return 0;
}

static int dense_inverse(r2p_cpr *P, const AmgLevel &C, hipStream_t s) {
    const int n = C.n;
    R2P_TRY(P->lu.ensure((size_t)n * n));
    R2P_TRY(P->luu.ensure((size_t)n * n));
    R2P_TRY(P->cinv.ensure((size_t)n * n));
    R2P_TRY(P->lupos.ensure(n));
    R2P_TRY(P->lurow.ensure(n));
    k_to_dense<<<n, BS, 0, s>>>(n, C.rp.p, C.col.p, C.val.p, P->lu.p, P->lupos.p, P->lurow.p);
    R2P_LAUNCH();
    // one workgroup holds a panel's rows: fewer columns where a thread holds
    // two or four rows
    if (n <= 256) R2P_TRY((dense_lu<256, 1, 32>(P, n, s)));
    else if (n <= 512) R2P_TRY((dense_lu<512, 1, 32>(P, n, s)));
    else if (n <= 1024) R2P_TRY((dense_lu<1024, 1, 32>(P, n, s)));
    else if (n <= 2048) R2P_TRY((dense_lu<1024, 2, 16>(P, n, s)));
    else R2P_TRY((dense_lu<1024, 4, 8>(P, n, s)));
    k_lu_gather<<<n, BS, 0, s>>>(n, P->lu.p, P->lurow.p, P->astatus.p, P->luu.p);
    R2P_LAUNCH();
#define R2P_INV(NR, AH) \
    k_dense_inv_col<NR, AH><<<n, 64, 0, s>>>(n, P->luu.p, P->lupos.p, P->astatus.p, P->cinv.p)
    // 64 NR >= n
    if (n <= 128) R2P_INV(2, 8);
    else if (n <= 256) R2P_INV(4, 6);
    else if (n <= 512) R2P_INV(8, 4);
    else if (n <= 1024) R2P_INV(16, 2);
    else
        k_dense_inv_col_lds<<<n, 64, sizeof(double) * n, s>>>(n, P->luu.p, P->lupos.p,
                                                            P->astatus.p, P->cinv.p);
#undef R2P_INV
    R2P_LAUNCH();
    return 0;
}

// ------------------------------------------------------- fused coarse levels
// Levels of up to FUSE_ROWS rows form the residual and its restriction in one
// kernel and the prolongation in the post-smoothing kernel: there a kernel is
// mostly its launch and a few dependent loads (3 to 4.5 us), so two kernels a
// level instead of four win, although the chains of loads get longer.  A cycle
// at 243,107 cells and five levels below: 182 us unfused, 171 with all levels
// fused (its largest, 82,086 rows, takes the same either way).  At 2M cells
// fusing the levels of 780,824 and 259,434 rows as well makes a solve 7%
// slower: such levels are bound by memory, and a fused kernel reads the rows
// in the order of the aggregates and gathers two vectors.
//
// A workgroup of the fused residual and restriction takes its members 64 at a
// time and rows longer than HEAVY four at a time, about 0.9 us each; where some
// workgroup has more than FUSE_STEPS such steps (k_fuse_steps), or an aggregate
// more than FEW members, the two run apart.  Levels of the benchmark's kind have
// up to 5 (4.5 to 8 us; apart 6 to 9 and a launch); hubs left by one matching
// round: 8,462 rows with an aggregate of 882 members 32 us, apart 8.
constexpr int FUSE_ROWS = 1 << 15;
constexpr int FUSE_STEPS = 5;
constexpr int CB = 256 / BIG;    // coarse rows of a workgroup of k_down_restrict

// Sets *slow (a pinned word) if a workgroup of k_down_restrict would take more
// than FUSE_STEPS steps.
__global__ __launch_bounds__(256) void k_fuse_steps(int nc, int nbs, const int *rp, const int *mptr,
                                                    const int *mem, const int *big, int *slow) {
    __shared__ int heavy, members;
    const int tid = threadIdx.x;
    int a, b, steps = 0;             // this thread's members: a, a + 256, .. below b
    if ((int)blockIdx.x < nbs) {
        int I = blockIdx.x * CB + tid / BIG;
        a = I < nc ? mptr[I] : 0;
        b = I < nc ? mptr[I + 1] : 0;
        if (b - a > BIG) b = a;
        a += tid % BIG;
    } else {
        int I = big[(int)blockIdx.x - nbs];
        a = mptr[I] + tid;
        b = mptr[I + 1];
    }
    for (bool more = true; more; a += 256) {
        if (tid == 0) heavy = members = 0;
        __syncthreads();
        if (a < b) {
            int i = mem[a];
            atomicAdd(&members, 1);
            if (rp[i + 1] - rp[i] > HEAVY) atomicAdd(&heavy, 1);
        }
        more = __syncthreads_or(a + 256 < b);
        steps += (members + 63) / 64 + (heavy + 3) / 4;
        __syncthreads();
    }
    if (tid == 0 && steps > FUSE_STEPS) *slow = 1;
}

// --------------------------------------------------------------- set-up
// Everything runs in order on one stream; the host waits only where it
// needs a count (the scans that return totals) and for the final status.
// Pinned words that kernels set, cleared (beside the one that takes the scans'
// totals): [0] for a list or row of more than FEW entries, [1] see k_fuse_steps.
// They are the host's to read once it has waited for a later scan.
static int hub_word(r2p_cpr *P, volatile int *&hub) {
    R2P_TRY(P->apin.ensure(64));
    hub = (volatile int *)P->apin.p + 8;
    hub[0] = hub[1] = 0;
    return 0;
}

// Member lists (CSR, ascending) of the nc aggregates of agg[0..n); uses two
// scratch arrays of n.  With *hub set, which the host sees after its next wait,
// only mptr is there (see sort_members).
static int build_members(r2p_cpr *P, int n, const int *agg, int nc, DBuf<int> &mptr,
                         DBuf<int> &mem, DBuf<int> &slot, DBuf<int> &list, volatile int *hub,
                         hipStream_t s) {
    R2P_TRY(mptr.ensure(nc + 1));
    R2P_TRY(mem.ensure(n));
    R2P_TRY(slot.ensure(n));
    R2P_TRY(list.ensure(n));
    int nb = r2p_blocks(n, BS);
    R2P_HIP(hipMemsetAsync(mptr.p, 0, sizeof(int) * (size_t)(nc + 1), s));
    k_member_slot<<<nb, BS, 0, s>>>(n, agg, mptr.p, slot.p);
    R2P_LAUNCH();
    R2P_TRY(r2p_scan_int(mptr.p, mptr.p, nc + 1, nullptr, P->aiscratch, P->apin, s));
    k_member_fill<<<nb, BS, 0, s>>>(n, agg, mptr.p, slot.p, list.p);
    R2P_LAUNCH();
    k_member_order<<<nb, BS, 0, s>>>(n, agg, mptr.p, list.p, mem.p, (int *)hub);
    R2P_LAUNCH();
    return 0;
}

// The lists' members by a stable sort of the rows by aggregate.
static int sort_members(r2p_cpr *P, int n, const int *agg, int nc, DBuf<int> &mem, hipStream_t s) {
    SetupWork &W = P->aws;
    DBuf<unsigned> &key = W.u[0], &kt = W.u[1], &vt = W.u[2];
    R2P_TRY(key.ensure(n));
    R2P_TRY(kt.ensure(n));
    R2P_TRY(vt.ensure(n));
    unsigned *val = (unsigned *)mem.p;
    k_member_keys<<<r2p_blocks(n, BS), BS, 0, s>>>(n, agg, key.p, val);
    R2P_LAUNCH();
    return r2p_sort_pairs(key.p, val, kt.p, vt.p, n, r2p_bits_for(nc), W.i[0], P->aiscratch,
                          P->apin, s);
}

// The product by sorting its terms.
static int galerkin_sorted(r2p_cpr *P, int n, int nnz, const int *rp, const int *col,
                           const double *val, const int *agg, int nc, DBuf<int> &rpc,
                           DBuf<int> &colc, DBuf<double> &valc, int *nnzc, hipStream_t s) {
    SetupWork &W = P->aws;
    DBuf<unsigned> &keyI = W.u[0], &keyJ = W.u[1], &keyS = W.u[2], &idx = W.u[3], &kt = W.u[4],
                   &vt = W.u[5];
    DBuf<int> &flag = W.i[0], &hist = W.i[1], &start = W.i[2];
    for (DBuf<unsigned> *b : {&keyI, &keyJ, &keyS, &idx, &kt, &vt}) R2P_TRY(b->ensure(nnz));
    R2P_TRY(flag.ensure(nnz + 1));
    k_gal_expand<<<r2p_blocks(n, BS / GS), BS, 0, s>>>(n, rp, agg, keyI.p, col, keyJ.p, idx.p);
    R2P_LAUNCH();
    const int bits = r2p_bits_for(nc), nb = r2p_blocks(nnz, BS);
    R2P_HIP(hipMemcpyAsync(keyS.p, keyJ.p, sizeof(unsigned) * (size_t)nnz, hipMemcpyDeviceToDevice, s));
    R2P_TRY(r2p_sort_pairs(keyS.p, idx.p, kt.p, vt.p, nnz, bits, hist, P->aiscratch, P->apin, s));
    k_gather_u<<<nb, BS, 0, s>>>(nnz, idx.p, keyI.p, keyS.p);
    R2P_LAUNCH();
    R2P_TRY(r2p_sort_pairs(keyS.p, idx.p, kt.p, vt.p, nnz, bits, hist, P->aiscratch, P->apin, s));
    // the coarse columns in sorted order (kt is free again)
    k_gather_u<<<nb, BS, 0, s>>>(nnz, idx.p, keyJ.p, kt.p);
    R2P_LAUNCH();
    k_gal_flags<<<nb, BS, 0, s>>>(nnz, keyS.p, kt.p, flag.p);
    R2P_LAUNCH();
    R2P_HIP(hipMemsetAsync(flag.p + nnz, 0, sizeof(int), s));
    int nnz_c = 0;
    R2P_TRY(r2p_scan_int(flag.p, flag.p, nnz + 1, &nnz_c, P->aiscratch, P->apin, s));
    R2P_TRY(colc.ensure(nnz_c));
    R2P_TRY(valc.ensure(nnz_c));
    R2P_TRY(start.ensure(nnz_c + 1));
    k_gal_runs<<<nb, BS, 0, s>>>(nnz, nc, keyS.p, kt.p, flag.p, start.p, rpc.p, nnz_c);
    R2P_LAUNCH();
    k_gal_sum<<<r2p_blocks(nnz_c, BS), BS, 0, s>>>(nnz_c, start.p, idx.p, kt.p, val, colc.p, valc.p);
    R2P_LAUNCH();
    *nnzc = nnz_c;
    return 0;
}

static int galerkin(r2p_cpr *P, int n, int nnz, const int *rp, const int *col, const double *val,
                    const int *agg, int nc, DBuf<int> &rpc, DBuf<int> &colc, DBuf<double> &valc,
                    int *nnzc, hipStream_t s) {
    SetupWork &W = P->aws;
    DBuf<int> &mptr = W.i[0], &mem = W.i[1], &slot = W.i[2], &list = W.i[3];
    DBuf<unsigned> &longs = W.u[0], &nlong = W.u[1];
    volatile int *hub;
    R2P_TRY(hub_word(P, hub));
    R2P_TRY(build_members(P, n, agg, nc, mptr, mem, slot, list, hub, s));
    R2P_TRY(longs.ensure(nc));
    R2P_TRY(nlong.ensure(1));
    R2P_TRY(rpc.ensure(nc + 1));
    R2P_HIP(hipMemsetAsync(nlong.p, 0, sizeof(int), s));
    GalArgs A;
    A.nc = nc;
    A.mptr = mptr.p; A.mem = mem.p; A.rp = rp; A.col = col; A.agg = agg; A.val = val;
    A.rpc = rpc.p; A.colc = nullptr; A.valc = nullptr;
    A.list = (int *)longs.p; A.nlist = (int *)nlong.p;
    A.hub = (int *)hub;
    const int nb = r2p_blocks(nc, 256 / GL), nl = std::min(nc, 1024);
    k_gal_rows<false><<<nb, 256, 0, s>>>(A);
    R2P_LAUNCH();
    k_gal_long<false><<<nl, 256, 0, s>>>(A);
    R2P_LAUNCH();
    int nnz_c = 0;
    R2P_TRY(r2p_scan_int(rpc.p, rpc.p, nc + 1, &nnz_c, P->aiscratch, P->apin, s));
    if (*hub) return galerkin_sorted(P, n, nnz, rp, col, val, agg, nc, rpc, colc, valc, nnzc, s);
    R2P_TRY(colc.ensure(nnz_c));
    R2P_TRY(valc.ensure(nnz_c));
    A.colc = colc.p; A.valc = valc.p;
    k_gal_rows<true><<<nb, 256, 0, s>>>(A);
    R2P_LAUNCH();
    k_gal_long<true><<<nl, 256, 0, s>>>(A);
    R2P_LAUNCH();
    *nnzc = nnz_c;
    return 0;
}

// One aggregation pass: agg (row -> aggregate) and the aggregate count.
static int aggregate_pass(r2p_cpr *P, int n, int nnz, const int *rp, const int *col,
                          const double *val, DBuf<int> &agg, int *nc, hipStream_t s) {
    SetupWork &W = P->aws;
    DBuf<double> &M = W.d[0], &wgt = W.d[1];
    DBuf<int> &match = W.i[0], &prop = W.i[1], &flag = W.i[2], &jt = W.i[3];
    R2P_TRY(M.ensure(n));
    R2P_TRY(wgt.ensure(nnz));
    R2P_TRY(match.ensure(n));
    R2P_TRY(prop.ensure(n));
    R2P_TRY(jt.ensure(n));
    R2P_TRY(flag.ensure(n + 1));
    int nb = r2p_blocks(n, BS), ng = r2p_blocks(n, BS / GS);
    double th = P->o.theta;
    k_weights<<<ng, BS, 0, s>>>(n, rp, col, val, wgt.p, M.p, match.p);
    R2P_LAUNCH();
    for (int r = 0; r < P->o.match_rounds; r++) {
        k_propose<<<ng, BS, 0, s>>>(n, rp, col, wgt.p, M.p, th, prop.p);
        R2P_LAUNCH();
        k_accept<<<nb, BS, 0, s>>>(n, prop.p, match.p, M.p);
        R2P_LAUNCH();
    }
    k_join<<<ng, BS, 0, s>>>(n, rp, col, wgt.p, M.p, th, jt.p);
    R2P_LAUNCH();
    k_leader_flag<<<nb, BS, 0, s>>>(n, match.p, jt.p, flag.p);
    R2P_LAUNCH();
    R2P_HIP(hipMemsetAsync(flag.p + n, 0, sizeof(int), s));
    int cnt = 0;
    R2P_TRY(r2p_scan_int(flag.p, flag.p, n + 1, &cnt, P->aiscratch, P->apin, s));
    R2P_TRY(agg.ensure(n));
    k_number<<<nb, BS, 0, s>>>(n, match.p, jt.p, flag.p, agg.p);
    R2P_LAUNCH();
    *nc = cnt;
    return 0;
}

// List (ascending) of the rows i < n with ptr[i+1] - ptr[i] > thr.
static int long_rows(r2p_cpr *P, int n, const int *ptr, int thr, DBuf<int> &list, int *count,
                     hipStream_t s) {
    DBuf<int> &flag = P->aws.i[0];
    R2P_TRY(flag.ensure(n + 1));
    k_long_flag<<<r2p_blocks(n + 1, BS), BS, 0, s>>>(n, ptr, thr, flag.p);
    R2P_LAUNCH();
    int cnt = 0;
    R2P_TRY(r2p_scan_int(flag.p, flag.p, n + 1, &cnt, P->aiscratch, P->apin, s));
    R2P_TRY(list.ensure(cnt));
    k_long_list<<<r2p_blocks(n, BS), BS, 0, s>>>(n, ptr, thr, flag.p, list.p);
    R2P_LAUNCH();
    *count = cnt;
    return 0;
}

int r2p_amg_setup(r2p_cpr *P, hipStream_t s) {
    r2p_jacobian *J = P->J;
    const Phys &ph = J->m->ph;
    int n = ph.n;
    AmgLevel &L0 = P->lv[0];
    // level 0 structure (static per model)
    if (P->app_n != n) {
        R2P_TRY(L0.rp.ensure(n + 1));
        k_app_count<<<r2p_blocks(n, BS), BS, 0, s>>>(ph, L0.rp.p);
        R2P_LAUNCH();
        R2P_HIP(hipMemsetAsync(L0.rp.p + n, 0, sizeof(int), s));
        int nnz = 0;
        R2P_TRY(r2p_scan_int(L0.rp.p, L0.rp.p, n + 1, &nnz, P->aiscratch, P->apin, s));
        R2P_TRY(L0.col.ensure(nnz));
        R2P_TRY(P->iscratch2.ensure(nnz));
        k_app_cols<<<r2p_blocks(n, BS), BS, 0, s>>>(ph, L0.rp.p, L0.col.p, P->iscratch2.p);
        R2P_LAUNCH();
        L0.n = n;
        L0.nnz = nnz;
        P->app_n = n;
    }
    R2P_TRY(L0.val.ensure(L0.nnz));
    k_app_vals<<<r2p_blocks(n, BS), BS, 0, s>>>(n, L0.rp.p, P->iscratch2.p, J->vp.p, L0.val.p);
    R2P_LAUNCH();
    R2P_TRY(L0.v7.ensure(7L * n));
    k_app_v7<<<r2p_blocks(7L * n, BS), BS, 0, s>>>(n, J->vp.p, L0.v7.p);
    R2P_LAUNCH();
    if (P->o.precision == R2P_FP32) {
        R2P_TRY(L0.v7f.ensure(7L * n));
        k_castv<float><<<r2p_blocks(7L * n, BS), BS, 0, s>>>(7L * n, L0.v7.p, L0.v7f.p);
        R2P_LAUNCH();
    }
    int maxlev = std::min(std::max(P->o.max_levels, 1), 24);
    int passes = std::max(P->o.agg_passes, 1);
    int l = 0;
    while (P->lv[l].n > P->o.max_coarse && l + 1 < maxlev) {
        AmgLevel &A = P->lv[l];
        AmgLevel &C = P->lv[l + 1];
        R2P_TRY(A.agg.ensure(A.n));
        k_iota<<<r2p_blocks(A.n, BS), BS, 0, s>>>(A.n, A.agg.p);
        R2P_LAUNCH();
        // successive passes, each on the Galerkin product of the previous one
        DBuf<int> *crp = P->aws.crp, *ccol = P->aws.ccol;
        DBuf<double> *cval = P->aws.cval;
        const int *rp = A.rp.p, *col = A.col.p;
        const double *val = A.val.p;
        int cn = A.n, nc = A.n, nnzc = 0, cnnz = A.nnz;
        for (int p = 0; p < passes; p++) {
            DBuf<int> &a = P->aws.agg;
            R2P_TRY(aggregate_pass(P, cn, cnnz, rp, col, val, a, &nc, s));
            bool last = p == passes - 1;
            DBuf<int> &orp = last ? C.rp : crp[p & 1];
            DBuf<int> &ocol = last ? C.col : ccol[p & 1];
            DBuf<double> &oval = last ? C.val : cval[p & 1];
            R2P_TRY(galerkin(P, cn, cnnz, rp, col, val, a.p, nc, orp, ocol, oval, &nnzc, s));
            cnnz = nnzc;
            k_compose<<<r2p_blocks(A.n, BS), BS, 0, s>>>(A.n, a.p, A.agg.p);
            R2P_LAUNCH();
            rp = orp.p; col = ocol.p; val = oval.p;
            cn = nc;
        }
        if (nc >= A.n) break;   // no coarsening progress
        C.n = nc;
        C.nnz = nnzc;
        volatile int *hub;
        R2P_TRY(hub_word(P, hub));
        R2P_TRY(build_members(P, A.n, A.agg.p, nc, A.mptr, A.mem, P->aws.i[0], P->aws.i[1], hub, s));
        R2P_TRY(long_rows(P, nc, A.mptr.p, BIG, A.big, &A.nbig, s));
        A.split = A.n > FUSE_ROWS || *hub != 0;
        if (*hub) R2P_TRY(sort_members(P, A.n, A.agg.p, nc, A.mem, s));
        if (l > 0 && !A.split) {
            int nbs = r2p_blocks(nc, CB);
            k_fuse_steps<<<nbs + A.nbig, 256, 0, s>>>(nc, nbs, A.rp.p, A.mptr.p, A.mem.p, A.big.p,
                                                      (int *)hub + 1);
            R2P_LAUNCH();
        }
        R2P_TRY(long_rows(P, nc, C.rp.p, HEAVY, C.heavy, &C.nheavy, s));
        A.split |= hub[1] != 0;
        l++;
    }
    P->nlev = l + 1;
    bool f32 = P->o.precision == R2P_FP32;
    for (int k = 0; k < P->nlev; k++) {
        AmgLevel &A = P->lv[k];
        R2P_TRY(A.l1.ensure(A.n));
        k_l1<<<r2p_blocks(A.n, BS), BS, 0, s>>>(A.n, A.rp.p, A.val.p, A.l1.p);
        R2P_LAUNCH();
        if (f32) {
            R2P_TRY(A.f32.val.ensure(A.nnz));
            R2P_TRY(A.f32.l1.ensure(A.n));
            R2P_TRY(A.bf.ensure(A.n));
            R2P_TRY(A.xf.ensure(A.n));
            R2P_TRY(A.xof.ensure(A.n));
            k_castv<float><<<r2p_blocks(A.nnz, BS), BS, 0, s>>>(A.nnz, A.val.p, A.f32.val.p);
            R2P_LAUNCH();
            k_castv<float><<<r2p_blocks(A.n, BS), BS, 0, s>>>(A.n, A.l1.p, A.f32.l1.p);
            R2P_LAUNCH();
        }
        R2P_TRY(A.b.ensure(A.n));
        R2P_TRY(A.x.ensure(A.n));
        R2P_TRY(A.xo.ensure(A.n));
        // K-cycle work vectors on the levels whose systems the K-cycle solves
        if (k >= 1 && k <= P->o.kcycle && k < P->nlev - 1) {
            if (f32) R2P_TRY(A.kvf.ensure(4L * A.n));
            else R2P_TRY(A.kv.ensure(4L * A.n));
            // partial pairs of the K-cycle products on this level (and of the
            // orthogonalisation pass, KO_BLOCKS at most)
            long nbk = r2p_blocks(A.n, BS / G) + r2p_blocks(A.nheavy, BS / 64);
            R2P_TRY(P->kpart.ensure(2 * std::max(nbk, (long)KO_BLOCKS)));
        }
    }
    R2P_TRY(P->kscal.ensure(4 * 24));
    // coarsest level: dense LU and inverse (FP64)
    AmgLevel &C = P->lv[P->nlev - 1];
    int nc = C.n;
    if (nc > 4096) {
        // coarsening stalled: a soft failure of the method (no dense solve of that size)
        r2p_set_error("AMG coarsening stalled: coarsest level of %d rows", nc);
        return R2P_NOT_CONVERGED;
    }
    P->ncoarse = nc;
    R2P_TRY(P->astatus.ensure(1));
    R2P_TRY(P->apin.ensure(64));
    R2P_HIP(hipMemsetAsync(P->astatus.p, 0, sizeof(int), s));
    R2P_TRY(dense_inverse(P, C, s));
    int *h = (int *)P->apin.p;
    R2P_HIP(hipMemcpyAsync(h, P->astatus.p, sizeof(int), hipMemcpyDeviceToHost, s));
    R2P_HIP(hipStreamSynchronize(s));
    if (*h) { r2p_set_error("coarsest AMG matrix is singular"); return R2P_ESINGULAR; }
    return 0;
}

// --------------------------------------------------------------- V-cycle
// Levels below the finest are CSR.  A group of G lanes takes one row (lanes
// stride over its entries two at a time, both requested before either is
// used, then a fixed butterfly), so a wavefront reads the entries of 64 / G
// consecutive rows contiguously; with about 8 entries per row every lane
// issues its loads at once.  Rows longer than HEAVY get a wavefront each in
// trailing workgroups, four entries per lane in flight.  The iterate every
// row reads is formed beforehand: the pre-smoothed x = b / d by the
// restriction that produces b, and the prolonged x + P xc by a pass over the
// fine rows, so each entry costs one gather.

template <class T>
struct CsrArgs {
    int n, nbs;                  // rows; workgroups of the G-lanes-per-row part
    const int *heavy;            // rows longer than HEAVY, one wavefront each
    int nheavy;
    const int *rp, *col;
    const T *val, *l1;
    const T *b;                  // right-hand side of this level
    const T *x;                  // iterate: pre-smoothed (down), prolonged (up)
    T *xo;                       // down: residual b - A x; up: x + (b - A x) / d
};

// The iterate a row's entries multiply: x itself, or x plus the coarse
// correction xc of the row's aggregate.
template <class T>
struct PlainX {
    const T *x;
    __device__ __forceinline__ T operator()(int j) const { return x[j]; }
};
template <class T>
struct ProlongedX {
    const T *x, *xc;
    const int *agg;
    __device__ __forceinline__ T operator()(int j) const { return x[j] + xc[agg[j]]; }
};

// Sum of entries z0 .. z1 of a row times the iterate: by a group of G lanes
// (lane0 of G, in every lane), and by a wavefront.
template <class T, class X>
__device__ __forceinline__ T row_sum(const CsrArgs<T> &A, int z0, int z1, int lane0, const X &x) {
    T acc = (T)0;
    for (int z = z0 + lane0; z < z1; z += 2 * G) {
        int zb = z + G < z1 ? z + G : z;
        int ca = A.col[z], cb = A.col[zb];
        T va = A.val[z], vb = A.val[zb];
        T xa = x(ca), xb = x(cb);
        acc += va * xa + (z + G < z1 ? vb * xb : (T)0);
    }
    acc += dpp_move<DPP_XOR1>(acc);
    acc += dpp_move<DPP_XOR2>(acc);
    return acc;
}
template <class T, class X>
__device__ __forceinline__ T row_sum_wave(const CsrArgs<T> &A, int z0, int z1, int lane, const X &x) {
    T acc = (T)0;
    for (int z = z0 + lane; z < z1; z += 256) {
        T t[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            int zz = z + 64 * u < z1 ? z + 64 * u : z;
            T v = A.val[zz] * x(A.col[zz]);
            t[u] = z + 64 * u < z1 ? v : (T)0;
        }
        acc += (t[0] + t[1]) + (t[2] + t[3]);
    }
    acc = wave_sum_up(acc);
    return acc;
}

// MODE: CSR_DOWN xo = b - A x; CSR_UP xo = x + (b - A x) / d; CSR_PRODUCT xo = A x.
enum { CSR_DOWN = 0, CSR_UP = 1, CSR_PRODUCT = 2 };
template <class T, int MODE, class X>
__device__ __forceinline__ void csr_level(const CsrArgs<T> &A, const X &x) {
    int i, lane0;
    T acc;
    if ((int)blockIdx.x < A.nbs) {
        i = xcd_block(blockIdx.x, A.nbs) * (blockDim.x / G) + (int)threadIdx.x / G;
        lane0 = threadIdx.x % G;
        if (i >= A.n) return;                 // whole groups leave together
        int z0 = A.rp[i], z1 = A.rp[i + 1];
        if (z1 - z0 > HEAVY) return;
        acc = row_sum(A, z0, z1, lane0, x);
    } else {
        int w = ((int)blockIdx.x - A.nbs) * (blockDim.x >> 6) + (threadIdx.x >> 6);
        if (w >= A.nheavy) return;
        lane0 = threadIdx.x & 63;
        i = A.heavy[w];
        acc = row_sum_wave(A, A.rp[i], A.rp[i + 1], lane0, x);
    }
    if (lane0 == 0)
        A.xo[i] = MODE == CSR_UP ? x(i) + (A.b[i] - acc) / A.l1[i]
                                 : (MODE == CSR_DOWN ? A.b[i] - acc : acc);
}
template <class T, int MODE>
__global__ __launch_bounds__(256) void k_csr_level(CsrArgs<T> A) {
    csr_level<T, MODE>(A, PlainX<T>{A.x});
}
// Post-smoothing with the prolongation in the same pass (see FUSE_ROWS).
template <class T>
__global__ __launch_bounds__(256) void k_csr_up(CsrArgs<T> A, const int *agg, const T *xc) {
    csr_level<T, CSR_UP>(A, ProlongedX<T>{A.x, xc, agg});
}

// Restriction P^T r: a group of GR lanes per coarse row (lanes stride over
// the members two at a time, then a fixed butterfly; aggregates average 2-4
// members);
// aggregates with more than BIG members (up to about a thousand on the
// coarse levels) get a wavefront each in trailing workgroups, four members
// per lane in flight.  When the coarse level is smoothed (xc given), its
// pre-smoothed iterate b / d is formed here.
constexpr int GR = 2;
template <class T>
__global__ __launch_bounds__(256) void k_restrict(int nc, int nbs, const int *mptr, const int *mem,
                                                  const int *big, int nbig, const T *r, T *bc,
                                                  const T *l1c, T *xc) {
    int I, lane0;
    T acc = (T)0;
    if ((int)blockIdx.x < nbs) {
        I = blockIdx.x * (blockDim.x / GR) + (int)threadIdx.x / GR;
        lane0 = threadIdx.x % GR;
        if (I >= nc) return;
        int a = mptr[I], b = mptr[I + 1];
        if (b - a > BIG) return;
        // two members per lane in flight
        for (int t = a + lane0; t < b; t += 2 * GR) {
            int tb = t + GR < b ? t + GR : t;
            int ma = mem[t], mb = mem[tb];
            T ra = r[ma], rb = r[mb];
            acc += ra + (t + GR < b ? rb : (T)0);
        }
        acc += dpp_move<DPP_XOR1>(acc);
    } else {
        int w = ((int)blockIdx.x - nbs) * (blockDim.x >> 6) + (threadIdx.x >> 6);
        if (w >= nbig) return;
        lane0 = threadIdx.x & 63;
        I = big[w];
        int a = mptr[I], b = mptr[I + 1];
        for (int t = a + lane0; t < b; t += 256) {
            T v[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                T rv = r[mem[t + 64 * u < b ? t + 64 * u : t]];
                v[u] = t + 64 * u < b ? rv : (T)0;
            }
            acc += (v[0] + v[1]) + (v[2] + v[3]);
        }
        acc = wave_sum_up(acc);
    }
    if (lane0 == 0) {
        bc[I] = acc;
        if (xc) xc[I] = acc / l1c[I];
    }
}

// Residual and restriction of a coarse level in one pass (see FUSE_ROWS):
// a workgroup takes CB coarse rows, whose members it lists in LDS, forms the
// members' residuals there (G lanes per row, rows longer than HEAVY by a
// wavefront) and adds them per coarse row in k_restrict's order.  An
// aggregate of more than BIG members takes a workgroup of its own, 256
// members at a time.
template <class T>
__device__ __forceinline__ void member_residuals(const CsrArgs<T> &A, const int *list, int cnt, T *res,
                                                 int *heavy, int *nheavy) {
    const PlainX<T> x{A.x};
    if (threadIdx.x == 0) *nheavy = 0;
    __syncthreads();
    for (int t = threadIdx.x / G; t < cnt; t += 256 / G) {
        int i = list[t], z0 = A.rp[i], z1 = A.rp[i + 1];
        if (z1 - z0 > HEAVY) {
            if (threadIdx.x % G == 0) heavy[atomicAdd(nheavy, 1)] = t;
            continue;
        }
        T r = A.b[i] - row_sum(A, z0, z1, threadIdx.x % G, x);
        if (threadIdx.x % G == 0) res[t] = r;
    }
    __syncthreads();
    for (int h = threadIdx.x / 64; h < *nheavy; h += 4) {
        int i = list[heavy[h]];
        T r = A.b[i] - row_sum_wave(A, A.rp[i], A.rp[i + 1], threadIdx.x & 63, x);
        if ((threadIdx.x & 63) == 0) res[heavy[h]] = r;
    }
    __syncthreads();
}

template <class T>
__global__ __launch_bounds__(256) void k_down_restrict(CsrArgs<T> A, int nc, int nbs, const int *mptr,
                                                       const int *mem, const int *big, T *bc,
                                                       const T *l1c, T *xc) {
    __shared__ int list[256], heavy[256], start[CB + 1], nheavy;
    __shared__ T res[256];
    const int tid = threadIdx.x;
    int I, lane0;
    T acc = (T)0;
    if ((int)blockIdx.x < nbs) {
        int I0 = xcd_block(blockIdx.x, nbs) * CB;
        // members of row tid / BIG, its place among the workgroup's
        I = I0 + tid / BIG;
        int a = I < nc ? mptr[I] : 0, cnt = I < nc ? mptr[I + 1] - a : 0;
        if (cnt > BIG) cnt = 0;
        if (tid % BIG == 0) start[tid / BIG] = cnt;
        __syncthreads();
        if (tid < 64) {
            int v = tid < CB ? start[tid] : 0, sum = v;
            for (int d = 1; d < CB; d <<= 1) {
                int u = __shfl_up(sum, d, 64);
                if (tid >= d) sum += u;
            }
            if (tid < CB) start[tid + 1] = sum;
            if (tid == 0) start[0] = 0;
        }
        __syncthreads();
        if (tid % BIG < cnt) list[start[tid / BIG] + tid % BIG] = mem[a + tid % BIG];
        member_residuals(A, list, start[CB], res, heavy, &nheavy);
        if (tid >= CB * GR) return;
        I = I0 + tid / GR;
        lane0 = tid % GR;
        int m0 = start[tid / GR], m1 = start[tid / GR + 1];
        for (int t = m0 + lane0; t < m1; t += 2 * GR) {
            T rb = t + GR < m1 ? res[t + GR] : (T)0;
            acc += res[t] + rb;
        }
        acc += dpp_move<DPP_XOR1>(acc);
        if (I >= nc || mptr[I + 1] - mptr[I] > BIG) return;
    } else {
        I = big[(int)blockIdx.x - nbs];
        lane0 = tid;
        int a = mptr[I], b = mptr[I + 1];
        for (int t = a; t < b; t += 256) {
            int cnt = min(256, b - t);
            if (tid < cnt) list[tid] = mem[t + tid];
            member_residuals(A, list, cnt, res, heavy, &nheavy);
            if (tid < cnt && tid < 64) {
                T v[4];
#pragma unroll
                for (int u = 0; u < 4; u++) v[u] = tid + 64 * u < cnt ? res[tid + 64 * u] : (T)0;
                acc += (v[0] + v[1]) + (v[2] + v[3]);
            }
            __syncthreads();
        }
        if (tid >= 64) return;
        acc = wave_sum_up(acc);
    }
    if (lane0 == 0) {
        bc[I] = acc;
        if (xc) xc[I] = acc / l1c[I];
    }
}

// Prolongation of the coarse correction onto a fine level's iterate:
// x_j += xc[agg_j], one thread per fine row.
template <class T>
__global__ void k_prolong(int n, const int *agg, const T *xc, T *x) {
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < n) x[j] = x[j] + xc[agg[j]];
}

// Level 0 in the 7-slot layout: columns are implied by the grid (clamped at
// the boundary, where the coefficient is 0) and summed in ascending order.
template <class T>
struct Level0 {
    int n, nx, nxy;
    const T *v7, *l1;
    const double *f;
    int fstride;
};

template <class T>
__global__ void k_down0(Level0<T> A, T *x, T *r) {
    int i = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    const int order[7] = {5, 3, 1, 0, 2, 4, 6};
    T bi = (T)A.f[(long)A.fstride * i];
    x[i] = bi / A.l1[i];
    T s = bi;
#pragma unroll
    for (int oi = 0; oi < 7; oi++) {
        int sl = order[oi];
        int j = i + slot_offset(sl, A.nx, A.nxy);
        j = j < 0 ? 0 : (j >= A.n ? A.n - 1 : j);
        s -= ld_stream(&A.v7[(long)sl * A.n + i]) * ((T)A.f[(long)A.fstride * j] / A.l1[j]);
    }
    r[i] = s;
}

// Post-smoothing of level 0 on the prolonged iterate x (= x + P xc).
// With ACC the result is added to xo (xo = xo + result, as a separate
// addition would) instead of replacing it.
template <class T, bool ACC>
__global__ void k_up0(Level0<T> A, const T *x, double *xo) {
    int i = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    const int order[7] = {5, 3, 1, 0, 2, 4, 6};
    T s = (T)A.f[(long)A.fstride * i];
#pragma unroll
    for (int oi = 0; oi < 7; oi++) {
        int sl = order[oi];
        int j = i + slot_offset(sl, A.nx, A.nxy);
        j = j < 0 ? 0 : (j >= A.n ? A.n - 1 : j);
        s -= ld_stream(&A.v7[(long)sl * A.n + i]) * x[j];
    }
    double v = (double)(x[i] + s / A.l1[i]);
    xo[i] = ACC ? xo[i] + v : v;
}

// Coarsest solve x = A_c^-1 b with the stored inverse (column-major, so a
// column read by 64 lanes is contiguous).  A workgroup of CS_WAVES
// wavefronts covers 64 rows; wavefront w sums its quarter of the columns,
// then the quarters are added in wavefront order.  A few workgroups in all, so
// bound by load latency: b is staged in LDS and COLS columns are in flight, a
// power of two that covers a wavefront's quarter up to 64 (412 rows: 12.3 us with
// 8 in flight and up to 7 left over one at a time, 8 with 64; 15 rows: 2.7 with
// 8, 4.6 with 64, most of them past the matrix).
constexpr int CS_WAVES = 4;
template <class T, int COLS>
__global__ __launch_bounds__(64 * CS_WAVES, 1) void k_coarse_solve(int n, const double *invT,
                                                                   const T *b, const double *f,
                                                                   int fstride, T *x, double *xd) {
    __shared__ double part[CS_WAVES][64];
    // n is at most 4,096, and 4 COLS below 64
    __shared__ double rhs[CS_WAVES][COLS < 64 ? 2 * COLS : 4096 / CS_WAVES + COLS];
    int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int i = blockIdx.x * 64 + lane;
    int q = (n + CS_WAVES - 1) / CS_WAVES;
    int c0 = w * q, cnt = min(n, c0 + q) - c0;
    int ii = i < n ? i : n - 1;
    // the wavefront's part of b, zeros behind it
    for (int c = lane; c < cnt + COLS; c += 64)
        rhs[w][c] = c < cnt ? (f ? f[(long)fstride * (c0 + c)] : (double)b[c0 + c]) : 0.0;
    // written by some lanes, read by others of the same wavefront, whose LDS
    // operations keep order
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    double s = 0.0, v[COLS];
    const double *col = invT + (long)c0 * n;
    for (int c = 0; c < cnt; c += COLS) {
#pragma unroll
        for (int u = 0; u < COLS; u++) {
            v[u] = col[ii];
            col += c + u + 1 < cnt ? n : 0;
        }
        __builtin_amdgcn_sched_barrier(0);    // all loads first
#pragma unroll
        for (int u = 0; u < COLS; u++) s += v[u] * rhs[w][c + u];
    }
    part[w][lane] = s;
    __syncthreads();
    if (w != 0 || i >= n) return;
    double t = part[0][lane];
    for (int k = 1; k < CS_WAVES; k++) t += part[k][lane];
    if (xd) xd[i] = t;
    else x[i] = (T)t;
}

// ------------------------------------------------------------- K-cycle
// Two generalised-conjugate-residual steps on a coarse level c (the
// corrections of the `kcycle` finest levels): p1 = C(b), q1 = A p1,
// a1 = (q1.b)/(q1.q1), r = b - a1 q1; p2 = C(r), q2 = A p2,
// beta = (q1.q2)/(q1.q1), p2 -= beta p1, q2 -= beta q1, a2 = (q2.r)/(q2.q2);
// the correction a1 p1 + a2 p2 is added by the prolongation.  The scalars
// stay on the device: the kernels that produce q1, q2 and the orthogonalised
// q2 also write per-workgroup partial sums of the dot products they feed,
// and one small workgroup adds the partials in workgroup order and forms
// the scalar, so nothing is read back and the sums do not depend on
// scheduling.

// Workgroup sum of (s0, s1) into part[blockIdx.x], part[gridDim.x + blockIdx.x].
__device__ __forceinline__ void block_partials(double s0, double s1, double *part) {
    __shared__ double red[2][BS / 64];
    s0 = wave_sum_down(s0);
    s1 = wave_sum_down(s1);
    int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) { red[0][wv] = s0; red[1][wv] = s1; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double t0 = 0.0, t1 = 0.0;
        for (int q = 0; q < BS / 64; q++) { t0 += red[0][q]; t1 += red[1][q]; }
        part[blockIdx.x] = t0;
        part[gridDim.x + blockIdx.x] = t1;
    }
}

// q = A p on a CSR level with the launch shape of k_csr_level (rows by
// groups of G lanes, rows longer than HEAVY by a wavefront in trailing
// workgroups), with per-workgroup partial dot products of q:
// DOT 0: (q.q, q.b); DOT 1: (q1.q, 0).
template <class T, int DOT>
__global__ __launch_bounds__(BS) void k_kspmv(CsrArgs<T> A, const T *q1, double *part) {
    double s0 = 0.0, s1 = 0.0;
    if ((int)blockIdx.x < A.nbs) {
        int i = xcd_block(blockIdx.x, A.nbs) * (BS / G) + (int)threadIdx.x / G;
        int lane0 = threadIdx.x % G;
        bool valid = i < A.n;
        int z0 = valid ? A.rp[i] : 0, z1 = valid ? A.rp[i + 1] : 0;
        bool heavy = z1 - z0 > HEAVY;
        T acc = row_sum(A, z0, heavy ? z0 : z1, lane0, PlainX<T>{A.x});
        if (lane0 == 0 && valid && !heavy) {
            A.xo[i] = acc;
            double q = (double)acc;
            if (DOT == 0) { s0 = q * q; s1 = q * (double)A.b[i]; }
            else s0 = (double)q1[i] * q;
        }
    } else {
        int w = ((int)blockIdx.x - A.nbs) * (BS / 64) + (int)(threadIdx.x >> 6);
        int lane = threadIdx.x & 63;
        if (w < A.nheavy) {
            int i = A.heavy[w];
            T acc = row_sum_wave(A, A.rp[i], A.rp[i + 1], lane, PlainX<T>{A.x});
            if (lane == 0) {
                A.xo[i] = acc;
                double q = (double)acc;
                if (DOT == 0) { s0 = q * q; s1 = q * (double)A.b[i]; }
                else s0 = (double)q1[i] * q;
            }
        }
    }
    block_partials(s0, s1, part);
}

// ks = {q1.q1, a1, beta, a2} from nb partial pairs: step 0 from
// (q1.q1, q1.b); 1 from q1.q2; 2 from (q2.q2, q2.r).  A zero denominator
// gives a zero step.
__global__ __launch_bounds__(1024) void k_kfin(int nb, const double *part, int step, double *ks) {
    __shared__ double red[2][1024 / 64];
    double s0 = 0.0, s1 = 0.0;
    // eight strides of partials requested together, then added in the same
    // order as one at a time (the result does not change)
    int st = blockDim.x, b = threadIdx.x;
    for (; b + 7 * st < nb; b += 8 * st) {
        double a0[8], a1[8];
#pragma unroll
        for (int u = 0; u < 8; u++) { a0[u] = part[b + u * st]; a1[u] = part[nb + b + u * st]; }
#pragma unroll
        for (int u = 0; u < 8; u++) { s0 += a0[u]; s1 += a1[u]; }
    }
    for (; b < nb; b += st) { s0 += part[b]; s1 += part[nb + b]; }
    s0 = wave_sum_down(s0);
    s1 = wave_sum_down(s1);
    int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) { red[0][wv] = s0; red[1][wv] = s1; }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double t0 = 0.0, t1 = 0.0;
    for (int q = 0; q < (int)(blockDim.x >> 6); q++) { t0 += red[0][q]; t1 += red[1][q]; }
    if (step == 0) {
        ks[0] = t0;
        ks[1] = t0 > 0.0 ? t1 / t0 : 0.0;
    } else if (step == 1) {
        ks[2] = ks[0] > 0.0 ? t0 / ks[0] : 0.0;
    } else {
        ks[3] = t0 > 0.0 ? t1 / t0 : 0.0;
    }
}

// r = b - a1 q1 (in place of b) and the next cycle's pre-smoothed iterate r / d.
template <class T>
__global__ void k_kres(int n, T *b, const T *q1, const double *ks, const T *l1, T *x) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    T r = (T)((double)b[i] - ks[1] * (double)q1[i]);
    b[i] = r;
    x[i] = r / l1[i];
}

// p2 -= beta p1, q2 -= beta q1, with partials of (q2.q2, q2.r) of the
// updated q2 (grid-stride over KO_BLOCKS workgroups).
template <class T>
__global__ __launch_bounds__(BS) void k_korth(int n, const T *p1, T *p2, const T *q1, T *q2,
                                              const T *r, const double *ks, double *part) {
    double beta = ks[2], s0 = 0.0, s1 = 0.0;
    for (int i = blockIdx.x * BS + threadIdx.x; i < n; i += gridDim.x * BS) {
        p2[i] = (T)((double)p2[i] - beta * (double)p1[i]);
        T q = (T)((double)q2[i] - beta * (double)q1[i]);
        q2[i] = q;
        s0 += (double)q * (double)q;
        s1 += (double)q * (double)r[i];
    }
    block_partials(s0, s1, part);
}

// Prolongation of the K-cycle correction: x_j += a1 p1[agg_j] + a2 p2[agg_j].
template <class T>
__global__ void k_prolong_k(int n, const int *agg, const T *p1, const T *p2, const double *ks,
                            T *x) {
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    int I = agg[j];
    T c = (T)(ks[1] * (double)p1[I] + ks[3] * (double)p2[I]);
    x[j] = x[j] + c;
}

// --------------------------------------------------------------- cycle
template <class T>
struct Cycle {
    r2p_cpr *P;
    hipStream_t s;
    int nl;
    bool acc = false;            // add the result to xp (hierarchies of two or more levels)
    static const T *vals(AmgLevel &A) {
        if constexpr (sizeof(T) == 4) return A.f32.val.p; else return (const T *)A.val.p;
    }
    static const T *l1s(AmgLevel &A) {
        if constexpr (sizeof(T) == 4) return A.f32.l1.p; else return (const T *)A.l1.p;
    }
    static T *vb(AmgLevel &A) {
        if constexpr (sizeof(T) == 4) return A.bf.p; else return (T *)A.b.p;
    }
    static T *vx(AmgLevel &A) {
        if constexpr (sizeof(T) == 4) return A.xf.p; else return (T *)A.x.p;
    }
    static T *vxo(AmgLevel &A) {
        if constexpr (sizeof(T) == 4) return A.xof.p; else return (T *)A.xo.p;
    }
    static T *kv(AmgLevel &A) {
        if constexpr (sizeof(T) == 4) return A.kvf.p; else return (T *)A.kv.p;
    }
    CsrArgs<T> csr(AmgLevel &A, const T *x, T *xo) {
        CsrArgs<T> a;
        a.n = A.n; a.nbs = r2p_blocks(A.n, BS / G);
        a.heavy = A.heavy.p; a.nheavy = A.nheavy;
        a.rp = A.rp.p; a.col = A.col.p; a.val = vals(A); a.l1 = l1s(A);
        a.b = vb(A);
        a.x = x; a.xo = xo;
        return a;
    }
    template <int MODE>
    int csr_launch(AmgLevel &A, const T *x, T *xo) {
        CsrArgs<T> D = csr(A, x, xo);
        k_csr_level<T, MODE><<<D.nbs + r2p_blocks(A.nheavy, BS / 64), BS, 0, s>>>(D);
        R2P_LAUNCH();
        return 0;
    }
    // Restriction of level l's residual (in its xo) to level l+1's right-hand
    // side, with l+1's pre-smoothed iterate when l+1 is smoothed.
    int restrict_to(int l) {
        AmgLevel &A = P->lv[l], &C = P->lv[l + 1];
        bool smooth = l + 1 < nl - 1;
        int nbs = r2p_blocks(C.n, BS / GR);
        k_restrict<T><<<nbs + r2p_blocks(A.nbig, BS / 64), BS, 0, s>>>(
            C.n, nbs, A.mptr.p, A.mem.p, A.big.p, A.nbig, vxo(A), vb(C),
            smooth ? l1s(C) : nullptr, smooth ? vx(C) : nullptr);
        R2P_LAUNCH();
        return 0;
    }
    // x = A_c^-1 b on the coarsest level, b in vb(C) or, stride fstride, in f.
    int coarse_solve(AmgLevel &C, const double *f, int fstride, T *x, double *xd) {
        const int q = (C.n + CS_WAVES - 1) / CS_WAVES;       // columns of a wavefront
#define R2P_CS(COLS) \
    k_coarse_solve<T, COLS><<<r2p_blocks(C.n, 64), 64 * CS_WAVES, 0, s>>>(C.n, P->cinv.p, vb(C), f, fstride, x, xd)
        if (q <= 8) R2P_CS(8);
        else if (q <= 16) R2P_CS(16);
        else if (q <= 32) R2P_CS(32);
        else R2P_CS(64);
#undef R2P_CS
        R2P_LAUNCH();
        return 0;
    }
    // The coarse correction of level l, added to level l's iterate vx(l).
    int correct(int l) {
        AmgLevel &A = P->lv[l], &C = P->lv[l + 1];
        int c = l + 1;
        if (l < P->o.kcycle && c < nl - 1) {
            int n = C.n;
            T *p1 = kv(C), *p2 = p1 + n, *q1 = p2 + n, *q2 = q1 + n;
            double *ks = P->kscal.p + 4 * c, *part = P->kpart.p;
            int nbs = r2p_blocks(n, BS / G), nbk = nbs + r2p_blocks(C.nheavy, BS / 64);
            int nbo = std::max(1, std::min(KO_BLOCKS, r2p_blocks(n, BS)));
            R2P_TRY(coarse(c, p1));
            k_kspmv<T, 0><<<nbk, BS, 0, s>>>(csr(C, p1, q1), nullptr, part);
            R2P_LAUNCH();
            k_kfin<<<1, 1024, 0, s>>>(nbk, part, 0, ks);
            R2P_LAUNCH();
            k_kres<T><<<r2p_blocks(n, BS), BS, 0, s>>>(n, vb(C), q1, ks, l1s(C), vx(C));
            R2P_LAUNCH();
            R2P_TRY(coarse(c, p2));
            k_kspmv<T, 1><<<nbk, BS, 0, s>>>(csr(C, p2, q2), q1, part);
            R2P_LAUNCH();
            k_kfin<<<1, 1024, 0, s>>>(nbk, part, 1, ks);
            R2P_LAUNCH();
            k_korth<T><<<nbo, BS, 0, s>>>(n, p1, p2, q1, q2, vb(C), ks, part);
            R2P_LAUNCH();
            k_kfin<<<1, 1024, 0, s>>>(nbo, part, 2, ks);
            R2P_LAUNCH();
            k_prolong_k<T><<<r2p_blocks(A.n, BS), BS, 0, s>>>(A.n, A.agg.p, p1, p2, ks, vx(A));
            R2P_LAUNCH();
        } else {
            R2P_TRY(coarse(c, vxo(C)));
            k_prolong<T><<<r2p_blocks(A.n, BS), BS, 0, s>>>(A.n, A.agg.p, vxo(C), vx(A));
            R2P_LAUNCH();
        }
        return 0;
    }
    // One cycle on a coarse (CSR) level c >= 1 whose right-hand side is in
    // vb(c) and, unless c is the coarsest, pre-smoothed iterate in vx(c);
    // the result goes to out.
    int coarse(int c, T *out) {
        AmgLevel &A = P->lv[c];
        if (c == nl - 1) {
            return coarse_solve(A, nullptr, 1, out, nullptr);
        }
        AmgLevel &C = P->lv[c + 1];
        const bool kc = c < P->o.kcycle && c + 1 < nl - 1;
        const bool smooth = c + 1 < nl - 1;
        if (!A.split) {
            int nbs = r2p_blocks(C.n, CB);
            k_down_restrict<T><<<nbs + A.nbig, BS, 0, s>>>(
                csr(A, vx(A), nullptr), C.n, nbs, A.mptr.p, A.mem.p, A.big.p, vb(C),
                smooth ? l1s(C) : nullptr, smooth ? vx(C) : nullptr);
            R2P_LAUNCH();
        } else {
            // the level's xo holds its residual until the correction is added
            R2P_TRY(csr_launch<CSR_DOWN>(A, vx(A), vxo(A)));
            R2P_TRY(restrict_to(c));
        }
        if (A.n > FUSE_ROWS || kc) {
            R2P_TRY(correct(c));
            return csr_launch<CSR_UP>(A, vx(A), out);
        }
        R2P_TRY(coarse(c + 1, vxo(C)));
        CsrArgs<T> D = csr(A, vx(A), out);
        k_csr_up<T><<<D.nbs + r2p_blocks(A.nheavy, BS / 64), BS, 0, s>>>(D, A.agg.p, vxo(C));
        R2P_LAUNCH();
        return 0;
    }
    // The cycle from level 0 (7-slot stencil) with right-hand side f (stride
    // fstride), result in xp.
    int run(const double *f, int fstride, double *xp) {
        if (nl == 1) {
            AmgLevel &C = P->lv[0];
            return coarse_solve(C, f, fstride, vx(C), xp);
        }
        const Phys &ph = P->J->m->ph;
        Level0<T> Z;
        AmgLevel &A = P->lv[0];
        Z.n = A.n; Z.nx = ph.nx; Z.nxy = ph.nx * ph.ny;
        if constexpr (sizeof(T) == 4) Z.v7 = A.v7f.p; else Z.v7 = (const T *)A.v7.p;
        Z.l1 = l1s(A);
        Z.f = f;
        Z.fstride = fstride;
        k_down0<T><<<r2p_blocks(A.n, BS), BS, 0, s>>>(Z, vx(A), vxo(A));
        R2P_LAUNCH();
        R2P_TRY(restrict_to(0));
        R2P_TRY(correct(0));
        if (acc)
            k_up0<T, true><<<r2p_blocks(Z.n, BS), BS, 0, s>>>(Z, vx(A), xp);
        else
            k_up0<T, false><<<r2p_blocks(Z.n, BS), BS, 0, s>>>(Z, vx(A), xp);
        R2P_LAUNCH();
        return 0;
    }
};

int r2p_amg_cycle(r2p_cpr *P, const double *f, int fstride, double *xp, hipStream_t s) {
    if (P->o.precision == R2P_FP32) {
        Cycle<float> c{P, s, P->nlev};
        return c.run(f, fstride, xp);
    }
    Cycle<double> c{P, s, P->nlev};
    return c.run(f, fstride, xp);
}

// r = f - A_pp xp on level 0 (the 7-slot stencil, summed as in k_up0), FP64.
template <class T>
__global__ void k_res0(Level0<T> A, const double *xp, double *r) {
    int i = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    const int order[7] = {5, 3, 1, 0, 2, 4, 6};
    double s = A.f[(long)A.fstride * i];
#pragma unroll
    for (int oi = 0; oi < 7; oi++) {
        int sl = order[oi];
        int j = i + slot_offset(sl, A.nx, A.nxy);
        j = j < 0 ? 0 : (j >= A.n ? A.n - 1 : j);
        s -= (double)ld_stream(&A.v7[(long)sl * A.n + i]) * xp[j];
    }
    r[i] = s;
}

// The pressure stage: amg_cycles cycles on A_pp xp = f_p from xp = 0, each
// on the residual of the last (xp = C(f_p), then xp = xp + C(f_p - A_pp xp)).
template <class T>
static int amg_apply_t(r2p_cpr *P, const double *f, int fstride, double *xp, hipStream_t s) {
    R2P_TRY(r2p_amg_cycle(P, f, fstride, xp, s));
    if (P->o.amg_cycles < 2 || P->nlev < 2) return 0;
    AmgLevel &A = P->lv[0];
    const Phys &ph = P->J->m->ph;
    Level0<T> Z;
    Z.n = A.n; Z.nx = ph.nx; Z.nxy = ph.nx * ph.ny;
    if constexpr (sizeof(T) == 4) Z.v7 = A.v7f.p; else Z.v7 = (const T *)A.v7.p;
    Z.l1 = nullptr;
    Z.f = f;
    Z.fstride = fstride;
    for (int k = 1; k < P->o.amg_cycles; k++) {
        k_res0<T><<<r2p_blocks(A.n, BS), BS, 0, s>>>(Z, xp, P->t_ares.p);
        R2P_LAUNCH();
        // the cycle's last kernel adds its result to xp
        Cycle<T> c{P, s, P->nlev};
        c.acc = true;
        R2P_TRY(c.run(P->t_ares.p, 1, xp));
    }
    return 0;
}

int r2p_amg_apply(r2p_cpr *P, const double *f, int fstride, double *xp, hipStream_t s) {
    if (P->o.precision == R2P_FP32) return amg_apply_t<float>(P, f, fstride, xp, s);
    return amg_apply_t<double>(P, f, fstride, xp, s);
}

extern "C" int r2p_amg_info(r2p_cpr *P, int level, int *nlev, int *n, int *nnz) {
    if (!P || !P->ready) { r2p_set_error("CPR not set up"); return R2P_ESTATE; }
    if (nlev) *nlev = P->nlev;
    if (level >= 0 && level < P->nlev) {
        if (n) *n = P->lv[level].n;
        if (nnz) *nnz = P->lv[level].nnz;
    }
    return 0;
}

extern "C" int r2p_amg_export_level(r2p_cpr *P, int level, int *rp, int *col, double *val,
                                    double *l1, int *agg, void *stream) {
    if (!P || !P->ready) { r2p_set_error("CPR not set up"); return R2P_ESTATE; }
    if (level < 0 || level >= P->nlev) { r2p_set_error("bad level"); return R2P_EINVAL; }
    R2P_HIP(hipStreamSynchronize((hipStream_t)stream));
    AmgLevel &A = P->lv[level];
    if (rp) R2P_HIP(hipMemcpy(rp, A.rp.p, sizeof(int) * (A.n + 1), hipMemcpyDeviceToHost));
    if (col) R2P_HIP(hipMemcpy(col, A.col.p, sizeof(int) * A.nnz, hipMemcpyDeviceToHost));
    if (val) R2P_HIP(hipMemcpy(val, A.val.p, sizeof(double) * A.nnz, hipMemcpyDeviceToHost));
    if (l1) R2P_HIP(hipMemcpy(l1, A.l1.p, sizeof(double) * A.n, hipMemcpyDeviceToHost));
    if (agg && level < P->nlev - 1)
        R2P_HIP(hipMemcpy(agg, A.agg.p, sizeof(int) * A.n, hipMemcpyDeviceToHost));
    return 0;
}
