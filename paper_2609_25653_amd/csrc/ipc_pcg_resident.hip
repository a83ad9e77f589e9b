// The whole PCG solve of a one-scene context in one launch.
//
// What bounds the launch-per-iteration form (k_pcg_step + k_spmv) on one
// scene is not the arithmetic: on the 20k-tet squeeze an iteration moves a
// few MB, yet takes 12 us, two launches of 5 us that are mostly start-up,
// dependent loads and drain; on the 200k-tet scene the product also reads the
// 45 MB matrix again every iteration (11.5 us of 23).  Here every workgroup
// keeps its rows of the matrix in registers (two blocks per lane) and LDS
// (the rest) for the whole solve, with its nodes' p, s, x and r, and only the
// vector z, the dot products' partials and the coarse sums travel.
//
// Exchange.  Workgroups exchange 8-byte words through memory with relaxed
// agent-scope atomics, which bypass the (per-XCD, mutually incoherent) L2s
// for these words alone: no fence, no write-back, no counter.  A word that
// has not been written yet holds PX_EMPTY, a NaN that no arithmetic makes, so
// a reader polls the very words it needs and the data's arrival is the
// synchronisation.  One iteration needs two exchanges (three with the coarse
// correction): the partials of r.z, r.r and z.Az to everybody, z to the rows
// that read it (and each domain's group sums to its workgroups).  256
// workgroups exchange the first two in 4.4 us, 80 in 3.1 us.
//   D  partials: three buffers; iteration k reads k % 3, writes (k + 1) % 3
//      and empties (k + 2) % 3.  A workgroup past its reads of iteration k
//      has seen every workgroup's partials of iteration k - 1's product, so
//      all have left the reads of iteration k - 1: the emptied buffer has no
//      reader left; and it stores its last partial of iteration k after its
//      emptying stores have completed, so whoever reads at k + 2 finds them.
//   Z, RC  (z; group sums): two buffers, written and read in iteration k
//      (k & 1), emptied in k + 1 by the same argument.
//
// Residency.  Every workgroup has to be running for the exchange to finish.
// The grid is at most the number of compute units, one workgroup fits on
// each, and one such launch per device runs at a time in this process.  A
// poll that waits longer than PX_WAIT (another process holding compute units)
// raises the abort word, every workgroup leaves, and the caller takes the
// launch-per-iteration form instead: the kernel writes nothing that form
// reads before its successful end.
//
// Bits.  Every sum runs in the order of k_spmv<8> and k_pcg_step<> (the same
// tiles, lanes, wavefront sums and partials), so both forms give the same
// iterates bit for bit.
//
// Split: T tiles of 64 rows per workgroup of 512 threads (8 lanes per row as
// in k_spmv<8>).  T = 1 as long as the tiles do not outnumber the compute
// units (more units share the LDS and register traffic), else 2, else 4; the
// coarse correction takes T = 4, which makes a workgroup one slice of a
// coarse domain.  T = 4 is what registers hold: 8 blocks per lane are 144 of
// the 256 registers.  Rows of more than LONG_ROW blocks go to workgroups of
// their own, as in k_spmv.
#include <mutex>

#include "ipc_device.h"
#include "ipc_internal.h"
#include "ipc_kernels.h"
#include "ipc_pcgdev.h"

namespace ipc {

typedef unsigned long long u64;
constexpr u64 PX_EMPTY = 0xFFF8DEADBEEFCAFEull;
constexpr int PX_NT = 512;                 // threads: a tile's 64 rows x 8 lanes
constexpr int PX_HALO = 1280;              // nodes of other workgroups a workgroup's short rows may read
constexpr int PX_HASH = 2048;              // their lookup table (set-up)
constexpr int PX_EXTRA = 2048;             // blocks past the two in registers, over all its short rows
constexpr int PX_EXTRA_LDS = 512;          // of these, kept in LDS (the others are read from memory)
constexpr int PX_BODIES = 16;              // affine bodies among a workgroup's nodes
constexpr int PX_VROWS = (PX_NT - 192) / 8 / 3;   // of these, with a coarse group: one row of 8 lanes per component
constexpr int PX_LONG = 512;               // long rows
constexpr long long PX_WAIT = 5000000;     // 50 ms of the 100 MHz clock

struct PxArgs {
    int N, ntile, G, nsp, nlong, nb, ncd, ndom, nfr, bnode0, maxit;
    const int *kind, *node_body, *row_ptr, *col, *dptr, *dcol, *long_rows, *node_da;
    const double *val, *dval, *dinv, *dinvB, *inv, *r0, *z0, *w0;
    const double *part, *part_zw, *part_long, *cg_part, *st;
    const int *act, *ph_ptr, *ph_e, *ph_n;
    double *x, *scal;
    int *iters, *ctl;
    u64 *D, *Z, *RC;
};

// words of one D buffer: r.z, r.r, z.Az per tile; z.Az per long row; r.z per
// coarse slice; A z of the long rows; A z of the bodies' translation nodes
__host__ __device__ inline int px_dlen(int ntile, int nlong, int ncd, int nb) { return 3 * ntile + 4 * nlong + ncd + 3 * nb; }

__device__ __forceinline__ u64 px_ld(const u64 *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void px_st(u64 *p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void px_put(u64 *p, double v) { px_st(p, (u64)__double_as_longlong(v)); }

// Poll the K words at the given places until none is empty.  Every wait
// ends: after PX_WAIT, or once any workgroup has given up (ctl[0]), the lane
// raises *gone and returns.
template <int K>
__device__ __forceinline__ void px_poll(const u64 *base, const unsigned (&at)[K], double (&v)[K], int *ctl, int *gone)
{
    u64 u[K];
    long long t0 = 0;
    for (int tries = 0;; ++tries) {
        bool miss = false;
#pragma unroll
        for (int i = 0; i < K; ++i) u[i] = px_ld(base + at[i]);
#pragma unroll
        for (int i = 0; i < K; ++i) miss |= u[i] == PX_EMPTY;
        if (!miss) break;
        if ((tries & 31) == 31) {
            const long long t = (long long)wall_clock64();
            if (t0 == 0) t0 = t;
            if (t - t0 > PX_WAIT) __hip_atomic_store(ctl, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (t - t0 > PX_WAIT || __hip_atomic_load(ctl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                *gone = 1;
                break;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < K; ++i) v[i] = __longlong_as_double((long long)u[i]);
}
// z of a node
__device__ __forceinline__ d3 px_poll3(const u64 *z, int node, int *ctl, int *gone)
{
    const unsigned o = 3u * (unsigned)node, q[3] = {o, o + 1, o + 2};
    double v[3];
    px_poll<3>(z, q, v, ctl, gone);
    return {v[0], v[1], v[2]};
}

// The three-term products of k_spmv and k_pcg_step, fused in the order that
// the compiler fuses them there; written out, because it chose another order
// for some of them here.
__device__ __forceinline__ double px_dot(double a0, double a1, double a2, d3 v)
{
    return __builtin_fma(a2, v.z, __builtin_fma(a0, v.x, a1 * v.y));
}
__device__ __forceinline__ double px_dt(d3 a, d3 v) { return px_dot(a.x, a.y, a.z, v); }
__device__ __forceinline__ d3 px_mat3v(const double *M, d3 v)
{
    return {px_dot(M[0], M[1], M[2], v), px_dot(M[3], M[4], M[5], v), px_dot(M[6], M[7], M[8], v)};
}
__device__ __forceinline__ void px_acc(const double *B, d3 w, double &ax, double &ay, double &az)
{
    ax += px_dot(B[0], B[1], B[2], w);
    ay += px_dot(B[3], B[4], B[5], w);
    az += px_dot(B[6], B[7], B[8], w);
}

// Shared memory of one workgroup.
template <int T>
struct PxLds {
    double zs[3 * (TILE * T + PX_HALO)];          // z: own nodes, then the halo
    double wv[3 * TILE * T];                      // A z of the own rows
    double px[6 * TILE * T];                      // p and x of the own nodes
    double eval[9 * PX_EXTRA_LDS];                // extra blocks
    double body[144 * PX_BODIES];                 // inverse blocks of the own bodies
    double rc[CG_N], zl[CG_ROWS], rcb[CG_N * PX_VROWS], zlb[3 * PX_VROWS + 1];
    double sh[3][8], shd[T][8], shl[3][8];
    int esrc[PX_EXTRA];                           // extra blocks: index into the matrix, or -1 - index into the pair-local blocks
    unsigned short eidx[PX_EXTRA];                // and their columns' places in zs
    int hkey[PX_HASH];
    unsigned short hslot[PX_HASH];
    int halo[PX_HALO];
    int lidx[TILE * T];                           // own node -> its long row, or -1
    int vdom[PX_VROWS], vgrp[PX_VROWS];           // own bodies with a coarse group: its domain and group
    short vof[TILE * T];                          // own node -> its entry there, or -1
    int nhalo, nextra, nbody, nv;
    int fit;                                      // raised in the set-up: the rows do not fit
    int gone[3];                                  // raised by a poll that gave up: phases scalars and long rows, coarse, halo
};

template <int T, bool COARSE>
__global__ void __launch_bounds__(PX_NT) k_pcg_resident(PxArgs A)
{
    extern __shared__ double px_smem[];
    PxLds<T> &S = *reinterpret_cast<PxLds<T> *>(px_smem);
    constexpr int OWN = TILE * T;
    const int tid0 = threadIdx.x, b = blockIdx.x;
    const bool tiles = b < A.G;                 // a workgroup of tiles, else one of long rows
    const int n0 = tiles ? b * OWN : 0;         // first own node
    const int dom = b / CG_SPLIT, sl = b % CG_SPLIT;
    const bool cg = COARSE && tiles && dom < A.ndom;
    const int DL = px_dlen(A.ntile, A.nlong, A.ncd, A.nb);
    const int oRR = A.ntile, oZW = 2 * A.ntile, oZL = 3 * A.ntile, oCG = oZL + A.nlong, oWL = oCG + A.ncd, oWB = oWL + 3 * A.nlong;

    int tid = tid0, lane = tid & (TILE - 1), wave = tid / TILE;
    // ---- set-up ---------------------------------------------------------------
    if (tid == 0) { S.nhalo = 0; S.nextra = 0; S.nbody = 0; S.nv = 0; S.fit = 0; S.gone[0] = S.gone[1] = S.gone[2] = 0; }
    for (int i = tid; i < PX_HASH; i += PX_NT) S.hkey[i] = -1;
    for (int i = tid; i < OWN; i += PX_NT) { S.lidx[i] = -1; S.vof[i] = -1; }
    __syncthreads();
    // the own nodes (threads 0 .. OWN - 1): n
    int n = n0 + tid;
    const bool own = tiles && tid < OWN && n < A.N;
    const int kd = own ? A.kind[n] : 2;
    const bool fem = kd == 0, bod = kd == 1;
    d3 rv = {0, 0, 0}, sv = {0, 0, 0};
    int ph = -1;          // COARSE: the body translation node that this padding slot stands for
    int bslot = 0;        // own body's place in S.body
    if (COARSE && cg && tid < OWN)
        for (int u = A.ph_ptr[dom]; u < A.ph_ptr[dom + 1]; ++u)
            if (A.ph_e[u] == sl * OWN + tid) ph = A.ph_n[u];
    if (own && kd != 2) {
        rv = ld3(A.r0, n);
        st3(S.zs, tid, ld3(A.z0, n));
        st3(S.wv, tid, ld3(A.w0, n));
    }
    if (ph >= 0) {
        rv = ld3(A.r0, ph);
        st3(S.wv, tid, ld3(A.w0, ph));
    }
    if (tid < OWN) {
        st3(S.px, tid, {0, 0, 0});
        st3(S.px, OWN + tid, {0, 0, 0});
        if (kd == 2) st3(S.zs, tid, {0, 0, 0});
    }
    if (bod) {
        // a body's 4 nodes are 4 lanes of one wavefront; the first takes the place
        const int a = n & 3;
        if (a == 0) bslot = atomicAdd(&S.nbody, 1);
        bslot = __shfl(bslot, lane - a);
        if (bslot >= PX_BODIES) S.fit = 2;
        else {
            const double *M = A.dinvB + 144 * (size_t)A.node_body[n - a] + 36 * a;
            for (int q = 0; q < 36; ++q) S.body[144 * bslot + 36 * a + q] = M[q];
        }
        if (COARSE && A.node_da[n] >= 0) {
            const int v = atomicAdd(&S.nv, 1);
            if (v >= PX_VROWS) S.fit = 2;
            else {
                S.vof[tid] = (short)v;
                S.vdom[v] = A.node_da[n] / CG_DOM;
                S.vgrp[v] = A.node_da[n] % CG_DOM;
            }
        }
    }
    for (int i = tid; i < A.nlong; i += PX_NT) {
        const int q = A.long_rows[i] - n0;
        if (tiles && q >= 0 && q < OWN) S.lidx[q] = i;
    }
    // the own rows (8 lanes each): collect the columns that other workgroups own
    int rk0[T], rk1[T], rd0[T], rd1[T];
    int sub = tid & 7;
#pragma unroll
    for (int j = 0; j < T; ++j) {
        const int r = n0 + TILE * j + tid / 8;
        rk0[j] = rk1[j] = rd0[j] = rd1[j] = 0;
        if (!tiles || r >= A.N) continue;
        const int k0 = A.row_ptr[r], k1 = A.row_ptr[r + 1], d0 = A.dptr[r], d1 = A.dptr[r + 1];
        if ((k1 - k0) + (d1 - d0) > LONG_ROW) continue;
        rk0[j] = k0; rk1[j] = k1; rd0[j] = d0; rd1[j] = d1;
        auto insert = [&](int c) {
            if (c >= n0 && c < n0 + OWN) return;
            unsigned h = ((unsigned)c * 2654435761u) >> 21;
            for (int probe = 0; probe < PX_HASH; ++probe, h = (h + 1) & (PX_HASH - 1)) {
                const int was = atomicCAS(&S.hkey[h], -1, c);
                if (was == c) return;
                if (was == -1) {
                    const int q = atomicAdd(&S.nhalo, 1);
                    if (q < PX_HALO) { S.hslot[h] = (unsigned short)(OWN + q); S.halo[q] = c; }
                    else S.fit = 2;
                    return;
                }
            }
            S.fit = 2;
        };
        for (int k = k0 + sub; k < k1; k += 8) insert(A.col[k]);
        for (int k = d0 + sub; k < d1; k += 8) insert(A.dcol[k]);
    }
    static_assert(PX_HASH == 2048, "the hash keeps 11 bits");
    __syncthreads();
    // blocks into registers (each lane's first two of a row), the others into the extra list
    double B[T][2][9];
    int bi[T], ex[T];   // places of the two columns; extra blocks: first | count << 16
    {
        auto place = [&](int c) -> int {
            if (c >= n0 && c < n0 + OWN) return c - n0;
            unsigned h = ((unsigned)c * 2654435761u) >> 21;
            for (int probe = 0; probe < PX_HASH; ++probe, h = (h + 1) & (PX_HASH - 1)) {
                if (S.hkey[h] == c) return S.hslot[h];
                if (S.hkey[h] == -1) break;
            }
            return 0;   // only after an overflow, which has raised S.fit
        };
        const bool ok = S.fit == 0;
#pragma unroll
        for (int j = 0; j < T; ++j) {
            bi[j] = 0;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int k = rk0[j] + sub + 8 * u;
                const bool in = ok && k < rk1[j];
                if (in) bi[j] |= place(A.col[k]) << (16 * u);
#pragma unroll
                for (int q = 0; q < 9; ++q) B[j][u][q] = in ? A.val[9 * (size_t)k + q] : 0.0;
            }
            const int ks = rk0[j] + sub + 16, ds = rd0[j] + sub;
            const int m = (ks < rk1[j] ? (rk1[j] - ks + 7) / 8 : 0) + (ds < rd1[j] ? (rd1[j] - ds + 7) / 8 : 0);
            int e = 0;
            ex[j] = 0;
            if (ok && m > 0) {
                e = atomicAdd(&S.nextra, m);
                if (e + m > PX_EXTRA) S.fit = 2;
                else {
                    ex[j] = e | m << 16;
                    int f = e;
                    for (int k = ks; k < rk1[j]; k += 8, ++f) { S.esrc[f] = k; S.eidx[f] = (unsigned short)place(A.col[k]); }
                    for (int k = ds; k < rd1[j]; k += 8, ++f) { S.esrc[f] = -1 - k; S.eidx[f] = (unsigned short)place(A.dcol[k]); }
                }
            }
        }
    }
    __syncthreads();
    for (int i = tid; i < 9 * min(S.nextra, PX_EXTRA_LDS); i += PX_NT) {
        const int s = S.esrc[i / 9];
        S.eval[i] = s >= 0 ? A.val[9 * (size_t)s + i % 9] : A.dval[9 * (size_t)(-1 - s) + i % 9];
    }
    // a long-row workgroup: its first row's first blocks, in the registers of the tiles' blocks
    int lrow = 0, lk = 0, lk1 = 0, ld = 0, ld1 = 0, lc[2] = {-1, -1};
    if (!tiles) {
        lrow = A.long_rows[b - A.G];
        const int k = A.row_ptr[lrow] + tid, d = A.dptr[lrow] + tid;
        lk1 = A.row_ptr[lrow + 1]; ld1 = A.dptr[lrow + 1];
        if (k < lk1) lc[0] = A.col[k];
        if (d < ld1) lc[1] = A.dcol[d];
        lk = k + PX_NT; ld = d + PX_NT;
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            B[0][0][q] = lc[0] >= 0 ? A.val[9 * (size_t)k + q] : 0.0;
            B[0][1][q] = lc[1] >= 0 ? A.dval[9 * (size_t)d + q] : 0.0;
        }
    }
    __syncthreads();
    if (S.fit) {   // does not fit: everybody leaves
        if (tid == 0) __hip_atomic_store(A.ctl, S.fit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }

    // ---- iterations -------------------------------------------------------------
    int a = A.act[0], itc = 0;
    double gam0 = 0.0, al0 = 0.0, eta2 = 0.0;
    const double eta = A.st[2];
    // Why a workgroup's threads leave together: a flag is raised only before
    // its phase's barrier (the long rows' polls share the next scalars') and
    // read only after it.
    bool indef = false, gone = false;
    const int li = own && kd != 2 ? S.lidx[tid] : -1;   // this node's row is a long one
    const int phb = ph >= 0 ? (ph - A.bnode0) / 4 : -1;
    for (int k = 0; a; ++k) {
        // the thread's number anew in every iteration: what is derived from it
        // is then formed where it is used instead of being kept in registers
        // that the blocks need
        tid = tid0;
        asm volatile("" : "+v"(tid));
        lane = tid & (TILE - 1); wave = tid / TILE; n = n0 + tid; sub = tid & 7;
        const u64 *Dk = A.D + (size_t)(k % 3) * DL;
        u64 *Dn = A.D + (size_t)((k + 1) % 3) * DL, *Dr = A.D + (size_t)((k + 2) % 3) * DL;
        u64 *Zk = A.Z + (size_t)(k & 1) * 3 * A.N, *Zr = A.Z + (size_t)((k + 1) & 1) * 3 * A.N;
        u64 *RCk = A.RC + (size_t)(k & 1) * CG_N * A.ndom, *RCr = A.RC + (size_t)((k + 1) & 1) * CG_N * A.ndom;
        d3 zv = {0, 0, 0};
        double Mi[9];   // read again every iteration (L2), behind the polls: the registers hold the blocks
        {
            const double *M = A.dinv + 9 * (size_t)(own ? n : 0);
#pragma unroll
            for (int q = 0; q < 9; ++q) Mi[q] = M[q];
        }
        // ---- the scalars: wavefronts 0-3 sum r.z and r.r, 4-7 z.Az (the sums of bs_finish) ----
        {
            const int t = tid & (BLOCK - 1);
            double v0 = 0.0, v1 = 0.0;
            if (k == 0) {   // from the launches before this one
                double e[2][4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = t + u * BLOCK;
                    const bool in = i < A.ntile;
                    e[0][u] = in ? (tid < BLOCK ? A.part[i] : A.part_zw[i]) : 0.0;
                    e[1][u] = in && tid < BLOCK ? A.part[A.ntile + i] : 0.0;
                }
                v0 = (e[0][0] + e[0][1]) + (e[0][2] + e[0][3]);
                v1 = (e[1][0] + e[1][1]) + (e[1][2] + e[1][3]);
                if (tid >= BLOCK) for (int i = t; i < A.nlong; i += BLOCK) v0 += A.part_long[i];
                else for (int i = t; i < A.ncd; i += BLOCK) v0 += A.cg_part[i];
            } else if (tid < BLOCK) {
                // lanes past the end poll the first tile's word and drop it; a
                // lane whose A z comes from a long row (or that stands for a
                // body node) polls it with the rest
                unsigned p[2 * T + 3];
                double e[2 * T + 3];
                const int far = li >= 0 ? oWL + 3 * li : phb >= 0 ? oWB + 3 * phb : -1;
#pragma unroll
                for (int u = 0; u < T; ++u) {
                    const int i = t + u * BLOCK;
                    p[2 * u] = i < A.ntile ? i : 0;
                    p[2 * u + 1] = p[2 * u] + oRR;
                }
#pragma unroll
                for (int q = 0; q < 3; ++q) p[2 * T + q] = far >= 0 ? far + q : 0;
                px_poll<2 * T + 3>(Dk, p, e, A.ctl, &S.gone[0]);
                if (far >= 0) st3(S.wv, tid, {e[2 * T], e[2 * T + 1], e[2 * T + 2]});
                double f[2][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
                for (int u = 0; u < T; ++u)
                    if (t + u * BLOCK < A.ntile) { f[0][u] = e[2 * u]; f[1][u] = e[2 * u + 1]; }
                v0 = (f[0][0] + f[0][1]) + (f[0][2] + f[0][3]);
                v1 = (f[1][0] + f[1][1]) + (f[1][2] + f[1][3]);
                if (COARSE)
                    for (int i = t; i < A.ncd; i += BLOCK) {
                        const unsigned q[1] = {(unsigned)(oCG + i)};
                        double c[1];
                        px_poll<1>(Dk, q, c, A.ctl, &S.gone[0]);
                        v0 += c[0];
                    }
            } else {
                unsigned p[T];
                double e[T], f[4] = {0, 0, 0, 0};
#pragma unroll
                for (int u = 0; u < T; ++u) p[u] = oZW + (t + u * BLOCK < A.ntile ? t + u * BLOCK : 0);
                px_poll<T>(Dk, p, e, A.ctl, &S.gone[0]);
#pragma unroll
                for (int u = 0; u < T; ++u)
                    if (t + u * BLOCK < A.ntile) f[u] = e[u];
                v0 = (f[0] + f[1]) + (f[2] + f[3]);
                for (int i = t; i < A.nlong; i += BLOCK) {
                    const unsigned q[1] = {(unsigned)(oZL + i)};
                    double c[1];
                    px_poll<1>(Dk, q, c, A.ctl, &S.gone[0]);
                    v0 += c[0];
                }
            }
            v0 = wave_sum(v0);
            if (tid < BLOCK) v1 = wave_sum(v1);
            if (lane == 0) { S.sh[0][wave] = v0; S.sh[1][wave] = v1; }
        }
        __syncthreads();
        if (S.gone[0]) { gone = true; break; }
        const double gam = (S.sh[0][0] + S.sh[0][1]) + (S.sh[0][2] + S.sh[0][3]);
        const double rr = (S.sh[1][0] + S.sh[1][1]) + (S.sh[1][2] + S.sh[1][3]);
        double del = (S.sh[0][4] + S.sh[0][5]) + (S.sh[0][6] + S.sh[0][7]);
        double be = 0.0;
        int na = 1;
        if (a == 2) {
            eta2 = eta * eta * rr;
            if (!(rr > 0.0)) na = 0;
        } else {
            if (rr <= eta2 || itc >= A.maxit) na = 0;
            else {
                be = gam / gam0;
                del -= be * gam / al0;
            }
        }
        if (na && !(del > 0.0)) { na = 0; indef = true; }
        if (!na) { a = 0; break; }
        const double al = gam / del;
        gam0 = gam; al0 = al; a = 1; ++itc;
        // ---- empty the words this workgroup writes next time ----
        if (tiles) {
            if (tid < T && n0 / TILE + tid < A.ntile) {
                const int t = n0 / TILE + tid;
                px_st(Dr + t, PX_EMPTY); px_st(Dr + oRR + t, PX_EMPTY); px_st(Dr + oZW + t, PX_EMPTY);
            }
            if (kd != 2)
#pragma unroll
                for (int q = 0; q < 3; ++q) px_st(Zr + 3 * (size_t)n + q, PX_EMPTY);
            if (COARSE) {
                if (cg && tid == T) px_st(Dr + oCG + CG_SPLIT * dom + sl, PX_EMPTY);
                if (cg && tid >= TILE && tid < TILE + CG_ROWS) px_st(RCr + (size_t)CG_N * dom + CG_ROWS * sl + tid - TILE, PX_EMPTY);
                if (bod && (n & 3) == 0 && li < 0)
#pragma unroll
                    for (int q = 0; q < 3; ++q) px_st(Dr + oWB + 3 * ((n - A.bnode0) / 4) + q, PX_EMPTY);
            }
        } else if (tid == 0) {
            for (int i = b - A.G; i < A.nlong; i += A.nsp) {
                px_st(Dr + oZL + i, PX_EMPTY);
                for (int q = 0; q < 3; ++q) px_st(Dr + oWL + 3 * i + q, PX_EMPTY);
                const int r = A.long_rows[i] - A.bnode0;
                if (COARSE && r >= 0 && (r & 3) == 0 && r / 4 < A.nb)
                    for (int q = 0; q < 3; ++q) px_st(Dr + oWB + 3 * (r / 4) + q, PX_EMPTY);
            }
        }
        // ---- the update of the own nodes (k_pcg_step) ----
        double rz = 0.0, rr1 = 0.0;
        if (tiles && tid < OWN) {
            if (kd != 2 || ph >= 0) pcg_sr(ld3(S.wv, tid), al, be, sv, rv);
            const d3 zo = ld3(S.zs, tid);
            if (fem) zv = px_mat3v(Mi, rv);
            else if (bod) {
                const int q4 = n & 3, first = lane - q4;
                double rb[12];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    rb[3 * q] = __shfl(rv.x, first + q);
                    rb[3 * q + 1] = __shfl(rv.y, first + q);
                    rb[3 * q + 2] = __shfl(rv.z, first + q);
                }
                // the sums of body_rows; one row's words in registers at a time
                const double *M = S.body + 144 * bslot + 36 * q4;
                double zz[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    double acc = 0.0;
#pragma unroll
                    for (int j = 0; j < 12; ++j) acc = __builtin_fma(M[12 * c + j], rb[j], acc);
                    zz[c] = acc;
                    asm volatile("" ::: "memory");
                }
                zv = {zz[0], zz[1], zz[2]};
            }
            if (kd != 2) {
                rr1 = px_dt(rv, rv);
                rz = px_dt(rv, zv);
                if (!COARSE) {
                    u64 *Zp = Zk + 3 * (size_t)n;
                    px_put(Zp, zv.x); px_put(Zp + 1, zv.y); px_put(Zp + 2, zv.z);
                    st3(S.zs, tid, zv);
                }
                d3 pv = ld3(S.px, tid), xv = ld3(S.px, OWN + tid);
                pv = {zo.x + be * pv.x, zo.y + be * pv.y, zo.z + be * pv.z};
                xv = {xv.x + al * pv.x, xv.y + al * pv.y, xv.z + al * pv.z};
                st3(S.px, tid, pv);
                st3(S.px, OWN + tid, xv);
            }
            if (COARSE && cg) {
                const d3 v = cg_group_sum(fem || ph >= 0 ? rv : d3{0, 0, 0});
                if ((lane & (CG_AGG - 1)) == CG_AGG - 1) {
                    u64 *p = RCk + (size_t)CG_N * dom + CG_ROWS * sl + 3 * (tid / CG_AGG);
                    px_put(p, v.x); px_put(p + 1, v.y); px_put(p + 2, v.z);
                }
            }
            rz = wave_sum(rz); rr1 = wave_sum(rr1);
            if (lane == 0 && n0 / TILE + wave < A.ntile) {
                px_put(Dn + n0 / TILE + wave, rz);
                px_put(Dn + oRR + n0 / TILE + wave, rr1);
            }
        }
        if (COARSE && tiles) {
            // the coarse correction: the rows of the domains' inverses (own
            // groups: threads 0-191; own bodies' groups: the others), from
            // the L2 while the group sums arrive: they would not fit the
            // registers beside the blocks
            const int crow = tid < 192 ? tid / CG_CLANES : (tid - 192) / CG_CLANES, cl = tid % CG_CLANES;
            const double *M = A.inv;
            if (tid < 192) M += (size_t)(cg ? dom : 0) * CG_N * CG_N + (size_t)(CG_ROWS * sl + crow) * CG_N;
            else if (crow / 3 < min(S.nv, PX_VROWS))
                M += (size_t)S.vdom[crow / 3] * CG_N * CG_N + (size_t)(3 * S.vgrp[crow / 3] + crow % 3) * CG_N;
            double m[CG_CPL];
#pragma unroll
            for (int j = 0; j < CG_CPL; ++j) m[j] = M[cl + CG_CLANES * j];
            for (int i = tid; i < (cg ? CG_N : 0) + CG_N * S.nv; i += PX_NT) {
                const int v = cg ? i / CG_N - 1 : i / CG_N;   // -1: the own domain
                const unsigned q[1] = {(unsigned)(CG_N * (v < 0 ? dom : S.vdom[v]) + i % CG_N)};
                double c[1];
                px_poll<1>(RCk, q, c, A.ctl, &S.gone[1]);
                if (v < 0) S.rc[i] = c[0];
                else S.rcb[CG_N * v + i % CG_N] = c[0];
            }
            __syncthreads();
            if (S.gone[1]) { gone = true; break; }
            if (tid < 192) {
                const double s = cg_row(m, S.rc, cl);
                if (cl == 0) S.zl[crow] = s;
            } else if (S.nv > 0) {
                const double s = cg_row(m, S.rcb + CG_N * min(crow / 3, PX_VROWS - 1), cl);
                if (cl == 0 && crow < 3 * S.nv) S.zlb[crow] = s;
            }
            __syncthreads();
            if (own && kd != 2) {
                if (cg && fem) zv = {zv.x + S.zl[3 * (tid / CG_AGG)], zv.y + S.zl[3 * (tid / CG_AGG) + 1], zv.z + S.zl[3 * (tid / CG_AGG) + 2]};
                else if (S.vof[tid] >= 0) {
                    const double *zl = S.zlb + 3 * S.vof[tid];
                    zv = {zv.x + zl[0], zv.y + zl[1], zv.z + zl[2]};
                }
                u64 *Zp = Zk + 3 * (size_t)n;
                px_put(Zp, zv.x); px_put(Zp + 1, zv.y); px_put(Zp + 2, zv.z);
                st3(S.zs, tid, zv);
            }
            if (cg && tid < TILE) {
                double dot = tid < CG_ROWS ? S.rc[CG_ROWS * sl + tid] * S.zl[tid] : 0.0;
                dot = wave_sum(dot);
                if (tid == 0) px_put(Dn + oCG + CG_SPLIT * dom + sl, dot);
            }
        }
        // ---- w = A z (k_spmv<8>) ----
        if (tiles) {
            for (int i = tid; i < S.nhalo; i += PX_NT) st3(S.zs, OWN + i, px_poll3(Zk, S.halo[i], A.ctl, &S.gone[2]));
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the emptying stores have completed
            __syncthreads();
            if (S.gone[2]) { gone = true; break; }
#pragma unroll
            for (int j = 0; j < T; ++j) {
                double ax = 0.0, ay = 0.0, az = 0.0;
                px_acc(B[j][0], ld3(S.zs, bi[j] & 0xffff), ax, ay, az);
                px_acc(B[j][1], ld3(S.zs, bi[j] >> 16), ax, ay, az);
                for (int e = ex[j] & 0xffff, e1 = e + (ex[j] >> 16); e < e1; ++e) {
                    const d3 zc = ld3(S.zs, S.eidx[e]);
                    if (e < PX_EXTRA_LDS) px_acc(S.eval + 9 * e, zc, ax, ay, az);
                    else {
                        const int s = S.esrc[e];
                        px_acc(s >= 0 ? A.val + 9 * (size_t)s : A.dval + 9 * (size_t)(-1 - s), zc, ax, ay, az);
                    }
                }
                ax = lane_sum<8>(ax); ay = lane_sum<8>(ay); az = lane_sum<8>(az);
                double dot = 0.0;
                const int q = TILE * j + tid / 8;
                if (sub == 0 && n0 + q < A.N && S.lidx[q] < 0) {
                    st3(S.wv, q, {ax, ay, az});
                    dot = px_dt(ld3(S.zs, q), {ax, ay, az});
                    if (COARSE) {
                        const int r = n0 + q - A.bnode0;
                        if (r >= 0 && (r & 3) == 0 && r / 4 < A.nb) {
                            u64 *p = Dn + oWB + 3 * (r / 4);
                            px_put(p, ax); px_put(p + 1, ay); px_put(p + 2, az);
                        }
                    }
                }
                dot = wave_sum(dot);
                if (lane == 0) S.shd[j][wave] = dot;
            }
            __syncthreads();
            if (tid < T && n0 / TILE + tid < A.ntile) {
                double t = S.shd[tid][0];
                for (int q = 1; q < 8; ++q) t += S.shd[tid][q];
                px_put(Dn + oZW + n0 / TILE + tid, t);
            }
        } else {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            for (int i = b - A.G; i < A.nlong; i += A.nsp) {
                int r = lrow, k0 = lk, k1 = lk1, d0 = ld, d1 = ld1;
                double ax = 0.0, ay = 0.0, az = 0.0;
                d3 zr;
                const u64 *const z = Zk;
                if (i == b - A.G) {   // the first blocks and the row's own z in one poll (absent ones poll the row's z too)
                    const unsigned p = 3u * (unsigned)(lc[0] >= 0 ? lc[0] : r), pd = 3u * (unsigned)(lc[1] >= 0 ? lc[1] : r),
                                   pr = 3u * (unsigned)r;
                    const unsigned q[9] = {p, p + 1, p + 2, pd, pd + 1, pd + 2, pr, pr + 1, pr + 2};
                    double v[9];
                    px_poll<9>(z, q, v, A.ctl, &S.gone[0]);
                    zr = {v[6], v[7], v[8]};
                    if (lc[0] >= 0) px_acc(B[0][0], {v[0], v[1], v[2]}, ax, ay, az);
                    for (; k0 < k1; k0 += PX_NT) px_acc(A.val + 9 * (size_t)k0, px_poll3(z, A.col[k0], A.ctl, &S.gone[0]), ax, ay, az);
                    if (lc[1] >= 0) px_acc(B[0][1], {v[3], v[4], v[5]}, ax, ay, az);
                } else {
                    r = A.long_rows[i];
                    k0 = A.row_ptr[r] + tid; k1 = A.row_ptr[r + 1];
                    d0 = A.dptr[r] + tid; d1 = A.dptr[r + 1];
                    zr = px_poll3(z, r, A.ctl, &S.gone[0]);
                    for (; k0 < k1; k0 += PX_NT) px_acc(A.val + 9 * (size_t)k0, px_poll3(z, A.col[k0], A.ctl, &S.gone[0]), ax, ay, az);
                }
                for (; d0 < d1; d0 += PX_NT) px_acc(A.dval + 9 * (size_t)d0, px_poll3(z, A.dcol[d0], A.ctl, &S.gone[0]), ax, ay, az);
                ax = wave_sum(ax); ay = wave_sum(ay); az = wave_sum(az);
                if (lane == 0) { S.shl[0][wave] = ax; S.shl[1][wave] = ay; S.shl[2][wave] = az; }
                __syncthreads();
                if (tid == 0) {
                    for (int q = 1; q < 8; ++q) { ax += S.shl[0][q]; ay += S.shl[1][q]; az += S.shl[2][q]; }
                    const d3 w = {ax, ay, az};
                    u64 *p = Dn + oWL + 3 * i;
                    px_put(p, ax); px_put(p + 1, ay); px_put(p + 2, az);
                    const int rb = r - A.bnode0;
                    if (COARSE && rb >= 0 && (rb & 3) == 0 && rb / 4 < A.nb) {
                        p = Dn + oWB + 3 * (rb / 4);
                        px_put(p, ax); px_put(p + 1, ay); px_put(p + 2, az);
                    }
                    px_put(Dn + oZL + i, px_dt(zr, w));
                }
                __syncthreads();
            }
        }
    }
    // ---- the end: x, and this workgroup's vote that it has reached it ----
    if (gone) {
        if (tid == 0) __hip_atomic_store(A.ctl, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    if (own && kd != 2) st3(A.x, n, ld3(S.px, OWN + tid));
    if (tid == 0) {
        if (b == 0) {
            A.iters[0] = itc;
            if (indef) A.scal[S_INDEF] = 1.0;
        }
        atomicAdd(A.ctl + 1, 1);
    }
}

// empties the exchange words and clears the control words
__global__ void __launch_bounds__(BLOCK) k_pcgx_fill(int64_t n, u64 *__restrict__ p, int *__restrict__ ctl)
{
    for (int64_t i = blockIdx.x * (int64_t)BLOCK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLOCK) p[i] = PX_EMPTY;
    if (blockIdx.x == 0 && threadIdx.x < 2) ctl[threadIdx.x] = 0;
}

// after the solve: 1 when every workgroup reached its end, 2 when one ran
// out of its time, 3 when the rows do not fit, to the host's progress word
__global__ void k_pcgx_end(int wgs, const int *__restrict__ ctl, unsigned int seq, u64 *__restrict__ out)
{
    const int s = ctl[0] == 0 && ctl[1] == wgs ? 1 : ctl[0] == 2 ? 3 : 2;
    out[0] = ((u64)seq << 32) | (unsigned int)s;
}

template <int T, bool COARSE>
static void px_launch(const PxArgs &A, int wgs, hipStream_t st)
{
    hipLaunchKernelGGL((k_pcg_resident<T, COARSE>), dim3(wgs), dim3(PX_NT), sizeof(PxLds<T>), st, A);
}

// tiles per workgroup and workgroups, or T = 0: not for this context
struct PxShape { int T = 0, G = 0, nsp = 0; };
static PxShape px_shape(const ipc_ctx *c)
{
    PxShape s;
    const int ntile = c->N / TILE, cu = c->n_cu;
    const bool coarse = c->coarse_on && c->n_cdom > 0;
    if (c->n_scenes != 1 || c->spmv_lanes != 8 || !c->use_graphs || c->prof || !c->pcg_fused || c->n_long > PX_LONG || !c->resident_ok) return s;
    if (coarse && (!c->cg_fusable || c->n_cdom * CG_SPLIT > BLOCK * 4)) return s;
    const int room = cu - std::min(c->n_long, 16);   // units left for tiles
    int T, G;
    if (coarse) {
        T = 4;
        G = std::max(CG_SPLIT * c->n_cdom, (ntile + T - 1) / T);
    } else {
        T = ntile <= std::min(room, BLOCK) ? 1 : ntile <= 2 * std::min(room, BLOCK) ? 2 : 4;
        G = (ntile + T - 1) / T;
    }
    if (G > room || ntile > T * BLOCK || G <= 0) return s;
    s.T = T; s.G = G; s.nsp = std::min(c->n_long, cu - G);
    return s;
}

// exchange words of a one-scene context of N nodes and NB bodies (0: none)
static size_t px_words(int n_scenes, int N, int NB)
{
    if (n_scenes != 1 || N / TILE > 4 * BLOCK) return 0;
    const int ndom = N / (CG_AGG * CG_DOM) + 1;
    return 3 * (size_t)px_dlen(N / TILE, PX_LONG, CG_SPLIT * ndom, NB) + 6 * (size_t)N + 2 * (size_t)CG_N * ndom;
}

size_t pcg_resident_bytes(int n_scenes, int N, int NB)
{
    const size_t w = px_words(n_scenes, N, NB);
    return w ? Arena::round(8 * w) + Arena::round(2 * sizeof(int)) : 0;
}

template <int T, bool COARSE>
static bool px_allow()
{
    return hipFuncSetAttribute((const void *)k_pcg_resident<T, COARSE>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)sizeof(PxLds<T>)) == hipSuccess;
}

// The exchange memory of a new context.  A workspace context takes it only
// when the plan's slack stays free for the requests of later calls, so that
// a workspace sized by an earlier plan serves as it did.
void pcg_resident_setup(ipc_ctx *c)
{
    const size_t w = px_words(c->n_scenes, c->N, c->NB);
    if (!w) return;
    if (c->ws.base) {
        const size_t need = pcg_resident_bytes(c->n_scenes, c->N, c->NB);
        if (c->ws.used + need + c->ws.size / 17 + (1 << 20) > c->ws.size) return;
    }
    int cu = 0;
    if (hipGetDevice(&c->device) != hipSuccess || hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess)
        return;
    c->n_cu = cu;
    if (!px_allow<1, false>() || !px_allow<2, false>() || !px_allow<4, false>() || !px_allow<4, true>()) return;
    // its sums are those of 8 lanes per row: the lanes stay at 8 unless a count is forced
    const int lanes = c->spmv_lanes;
    if (!c->spmv_lanes_forced) c->spmv_lanes = 8;
    c->resident_ok = true;
    c->resident_ok = px_shape(c).T > 0;
    if (!c->resident_ok) {
        c->spmv_lanes = lanes;
        return;
    }
    c->d.px_words.alloc(w);
    c->d.px_ctl.alloc(2);
}

static std::mutex g_resident_mu[64];   // one resident solve per device at a time

bool pcg_resident(ipc_ctx *c, double *x)
{
    const PxShape s = px_shape(c);
    if (!s.T) return false;
    if (c->resident_skip > 0) { --c->resident_skip; return false; }
    Dev &D = c->d;
    if (!D.px_words.p) return false;
    // workgroups of two resident launches could each hold compute units the
    // other waits for; the lock is kept until this one's end is known
    std::unique_lock<std::mutex> lock(g_resident_mu[c->device & 63], std::try_to_lock);
    if (!lock.owns_lock()) return false;
    hipStream_t st = c->stream;
    PxArgs A{};
    const bool coarse = c->coarse_on && c->n_cdom > 0;
    A.N = c->N; A.ntile = c->N / TILE; A.G = s.G; A.nsp = s.nsp; A.nlong = c->n_long; A.nb = c->NB;
    A.ncd = coarse ? CG_SPLIT * c->n_cdom : 0;
    A.ndom = coarse ? c->n_cdom : 0; A.nfr = c->cg_nfr; A.bnode0 = c->sc[0].bnode0; A.maxit = c->sc[0].max_pcg;
    A.kind = D.node_kind.p; A.node_body = D.node_body.p; A.row_ptr = D.row_ptr.p; A.col = D.col.p; A.dptr = D.dyn_ptr.p; A.dcol = D.dyn_col.p;
    A.long_rows = D.long_rows.p; A.node_da = D.cg_node_da.p;
    A.val = D.val.p; A.dval = D.dyn_val.p; A.dinv = D.dinv.p; A.dinvB = D.dinvB.p; A.inv = D.cg_inv.p;
    A.r0 = D.r.p; A.z0 = D.z.p; A.w0 = D.w.p;
    A.part = D.pcg_part.p; A.part_zw = D.part_node3.p; A.part_long = D.part_long.p; A.cg_part = D.cg_part.p; A.st = D.pcg_st.p; A.act = D.pcg_act.p;
    A.ph_ptr = D.cg_ph_ptr.p; A.ph_e = D.cg_ph_e.p; A.ph_n = D.cg_ph_n.p;
    A.x = x; A.scal = D.scal.p; A.iters = D.pcg_iters.p; A.ctl = D.px_ctl.p;
    const int64_t nd = 3 * (int64_t)px_dlen(A.ntile, A.nlong, A.ncd, A.nb), nz = 6 * (int64_t)A.N, nr = 2 * (int64_t)CG_N * A.ndom;
    A.D = D.px_words.p; A.Z = A.D + nd; A.RC = A.Z + nz;
    const int wgs = s.G + s.nsp;
    hipLaunchKernelGGL(k_pcgx_fill, dim3(std::min(blocks_for(nd + nz + nr), 1024)), dim3(BLOCK), 0, st, nd + nz + nr, A.D, A.ctl);
    switch (s.T) {
    case 1: px_launch<1, false>(A, wgs, st); break;
    case 2: px_launch<2, false>(A, wgs, st); break;
    default:
        if (coarse) px_launch<4, true>(A, wgs, st);
        else px_launch<4, false>(A, wgs, st);
    }
    IPC_HIP(hipGetLastError());
    const unsigned int seq = pcg_next_seq(c);
    hipLaunchKernelGGL(k_pcgx_end, dim3(1), dim3(1), 0, st, wgs, D.px_ctl.p, seq, c->h_peek_dev);
    const int status = pcg_await(c, 0, seq, 1);
    if (status == 1) { ++c->resident_solves; return true; }
    c->resident_skip = status == 3 ? 256 : 64;   // the launch-per-iteration form for a while
    return false;
}

} // namespace ipc
