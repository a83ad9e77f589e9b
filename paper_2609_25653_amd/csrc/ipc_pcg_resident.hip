// The whole PCG solve of a context in one launch (a batch's scenes: at most
// two), each scene to its own end.
//
// What bounds the launch-per-iteration form (k_pcg_step + k_spmv) is not the
// arithmetic: on the 20k-tet squeeze an iteration moves a few MB, yet takes 12
// us, two launches of 5 us that are mostly start-up, dependent loads and drain;
// on the 200k-tet scene the product also reads the 45 MB matrix again every
// iteration (11.5 us of 23).  Here every workgroup keeps its rows of the matrix
// in registers (two blocks per lane) and LDS (the rest) for the whole solve,
// with its nodes' p, s, x and r, and only the vector z, the dot products'
// partials and the coarse sums travel.
//
// Measured, us per iteration, that form and this one: 625-tet block 8.5 and
// 3.9, most of it two exchanges; 20k-tet squeeze 12-14 and 6.4 (the body rows' chain: z -> poll -> sum -> partial -> poll);
// 200k tets, coarse, 22-23 and 12.3, or 16 once a workgroup's rows have 2000
// contact blocks, most of them read from memory again in every iteration.
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
// The grid is at most the number of compute units that the stream may use,
// one workgroup fits on each, and one such launch per device runs at a time in
// this process.  A poll that waits longer than PX_WAIT (another process
// holding compute units) raises the abort word, every workgroup leaves, and
// the solve starts again in the launch-per-iteration form, which sets again
// all that this kernel writes.  Two contexts stepping the 20k-tet squeeze at
// once, ms a step each, that form and this one: threads of one process 26.0
// and 20.8, processes 25.2 and 15.9 (no wait ran out), alone 23.2 and 13.9.
//
// Bits.  Every sum runs in the order of k_spmv<8> and k_pcg_step<> (the same
// tiles, lanes, wavefront sums and partials), so both forms give the same
// iterates bit for bit.
//
// Split: T tiles of 64 rows per workgroup of 512 threads.  T = 1 as long as the tiles do not outnumber the compute
// units (more units share the LDS and register traffic), else 2, else 4; the
// coarse correction takes T = 4, which makes a workgroup one slice of a
// coarse domain.  T = 4 is the most that the registers take: 8 blocks per lane
// are 144 of the 256, and 12 more (6 with the coarse correction) are spilled,
// 28 bytes of scratch memory per lane; T = 1 and 2 take 146 and 172 registers.
// The arguments and what follows from them do not fit the scalar registers
// (115 to 212 of them are kept in lanes of vector registers).  Rows of more
// than LONG_ROW blocks go to workgroups of their own, as in k_spmv.
#include <mutex>

#include "ipc_device.h"
#include "ipc_internal.h"
#include "ipc_kernels.h"
#include "ipc_pcgdev.h"

namespace ipc {

typedef unsigned long long u64;
constexpr u64 PX_EMPTY = 0xFFF8DEADBEEFCAFEull;
constexpr int PX_NT = 512;                 // threads: a tile's 64 rows x 8 lanes
constexpr int PX_HALO = 1024;              // nodes of other workgroups a workgroup's short rows may read
constexpr int PX_HASH = 2048;              // their lookup table (set-up)
constexpr int PX_BODIES = 16;              // affine bodies among a workgroup's nodes
constexpr int PX_EXTRA = 3840;             // blocks past the two in registers, over all its short rows: the first 512 in
                                           // registers too, one per thread,
constexpr int PX_POOL = 128;               // the next ones in LDS, the others read from memory,
constexpr int PX_CHUNK = 2 * PX_NT;        // and added to their rows this many at a time
constexpr int PX_VROWS = (PX_NT - 192) / 8 / 3;   // of these, with a coarse group: one row of 8 lanes per component
constexpr int PX_LONG = 512;               // long rows per scene (on average)
constexpr int PX_SPARE = 16;               // workgroups kept free of tiles for them
constexpr int PX_WGMAX = 256;              // workgroups per launch (compute units)
constexpr long long PX_WAIT = 5000000;     // 50 ms of the 100 MHz clock

// A scene's ranges: nodes, tiles, coarse domains, bodies, first body node
struct PxScene { int node0, ntile, tile0, dom0, ndom, body0, nb, bnode0, maxit; };
// A workgroup's part: its scene; tiles T tile .. T tile + T - 1 of it, or
// (tile < 0) long rows spare, spare + nsp, ... of it
struct PxPart { int scene, tile, spare, nsp; };
// All scenes' arrays; the kernel moves them to its scene's part first.
struct PxArgs {
    int N, ntile, nlong, nb, ncd, ndom, ndom_all, bnode0, maxit;
    const PxScene *scene;
    const PxPart *wg;
    const int *seg_long, *kind, *node_body, *row_ptr, *col, *dptr, *dcol, *long_rows, *node_da;
    const double *val, *dval, *dinv, *dinvB, *inv, *r0, *z0, *w0;
    const double *part, *part_rr, *part_zw, *part_long, *cg_part, *st;
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
// The abort word (ctl[0]): 0, 1 a wait was given up, 2 the rows of a workgroup
// do not fit.  It only grows: workgroups that leave because the word is up
// raise it too, and must not turn a 2 into a 1.
__device__ __forceinline__ void px_abort(int *ctl, int why) { (void)__hip_atomic_fetch_max(ctl, why, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Poll the words ld(0) .. ld(K - 1) until none that is needed is empty.
// Every wait ends: after PX_WAIT, or once any workgroup has given up
// (ctl[0]), the lane raises *gone and returns.
template <int K, class Ld, class Need>
__device__ __forceinline__ void px_poll(Ld ld, Need need, double (&v)[K], int *ctl, int *gone)
{
    u64 u[K];
    long long t0 = 0;
    for (int tries = 0;; ++tries) {
        bool miss = false;
#pragma unroll
        for (int i = 0; i < K; ++i) u[i] = px_ld(ld(i));
#pragma unroll
        for (int i = 0; i < K; ++i) miss |= need(i) && u[i] == PX_EMPTY;
        if (!miss) break;
        if ((tries & 31) == 31) {
            const long long t = (long long)wall_clock64();
            if (t0 == 0) t0 = t;
            if (t - t0 > PX_WAIT) px_abort(ctl, 1);
            if (t - t0 > PX_WAIT || __hip_atomic_load(ctl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                *gone = 1;
                break;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < K; ++i) v[i] = need(i) ? __longlong_as_double((long long)u[i]) : 0.0;
}
__device__ __forceinline__ double px_poll1(const u64 *p, int *ctl, int *gone)
{
    double v[1];
    px_poll<1>([&](int) { return p; }, [](int) { return true; }, v, ctl, gone);
    return v[0];
}
// z of a node
__device__ __forceinline__ d3 px_poll3(const u64 *z, int node, int *ctl, int *gone)
{
    const u64 *const p = z + 3u * (unsigned)node;
    double v[3];
    px_poll<3>([&](int i) { return p + i; }, [](int) { return true; }, v, ctl, gone);
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
    double zs[3 * (TILE * T + PX_HALO + 1)];      // z: own nodes, then the halo, then a zero
    double wv[3 * TILE * T];                      // A z of the own rows
    double px[12 * TILE * T];                     // p, x, r and s of the own nodes
    union {                                       // (by turns, with barriers between)
        double res[3 * (PX_CHUNK + 1)];           // a chunk of the extra blocks times z, then a zero
        double rcb[CG_N * PX_VROWS];              // group sums of the own bodies' domains
    };
    double pool[9 * PX_POOL];                     // extra blocks 512 ...
    double body[144 * PX_BODIES];                 // inverse blocks of the own bodies
    double rc[CG_N], zl[CG_ROWS], zlb[3 * PX_VROWS + 1];
    double sh[3][8], shd[T][8], shl[3][8];
    union {
        double mi[9 * TILE * T];                  // inverse diagonal blocks of the own nodes
        struct {
            int key[PX_HASH];
            unsigned short slot[PX_HASH];
        } h;                                      // set-up only: columns of other workgroups and their places in zs
    };
    int esrc[PX_EXTRA];                               // extra blocks: index into the matrix, or -1 - index into the pair-local blocks
    unsigned short eidx[PX_EXTRA];                    // and their columns' places in zs (bytes)
    int halo[PX_HALO];
    int lidx[TILE * T];                           // own node -> where its A z travels in D (a long row, or the
                                                  // body node that its slot stands for), or -1
    int vdom[PX_VROWS], vgrp[PX_VROWS];           // own bodies with a coarse group: its domain and group
    short vof[TILE * T];                          // own node -> its entry there, or -1
    unsigned char kind[TILE * T], bslot[TILE * T];   // own node: 0 FEM, 1 body, 2 none, 3 stands for a body's node; its body's place
    int nhalo, nextra, nbody, nv;
    int fit;                                      // raised in the set-up: the rows do not fit
    int gone[4];                                  // raised by a poll that gave up: phases scalars, coarse, halo, long rows
};

static_assert(sizeof(PxLds<4>) <= 160 * 1024 && sizeof(PxLds<1>) > 80 * 1024, "one workgroup per compute unit");

// The scalars of iteration k, alike in every thread of every workgroup: the
// sums of bs_finish (wavefronts 0-3: r.z, 4-7: z.Az and r.r), alpha, beta and
// the stop.  far: where this lane's node's A z travels in D (-1: nowhere);
// it is polled with the rest.  Returns whether the wait was given up;
// afterwards st.a is 0 when the solve has ended.
struct PxState {
    int a = 0, it = 0;
    double eta = 0.0, eta2 = 0.0, gam = 0.0, al = 0.0;
    bool indef = false;
};
template <int T>
__device__ __forceinline__ bool px_scalars(const PxArgs &A, PxLds<T> &S, PxState &st, int k, int tid, int far, double &al, double &be)
{
    const int lane = tid & (TILE - 1), wave = tid / TILE;
    const int DL = px_dlen(A.ntile, A.nlong, A.ncd, A.nb);
    const int oRR = A.ntile, oZW = 2 * A.ntile, oZL = 3 * A.ntile, oCG = oZL + A.nlong;
    const u64 *Dk = A.D + (size_t)(k % 3) * DL;
    {
        const int t = tid & (BLOCK - 1);
        const bool lo = tid < BLOCK;
        double v0, v1 = 0.0;
        if (k == 0) {   // from the launches before this one
            double e[2][4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = t + u * BLOCK;
                const bool in = i < A.ntile;
                e[0][u] = in ? (lo ? A.part[i] : A.part_zw[i]) : 0.0;
                e[1][u] = in && !lo ? A.part_rr[i] : 0.0;
            }
            v0 = (e[0][0] + e[0][1]) + (e[0][2] + e[0][3]);
            v1 = (e[1][0] + e[1][1]) + (e[1][2] + e[1][3]);
            if (lo) for (int i = t; i < A.ncd; i += BLOCK) v0 += A.cg_part[i];
            else for (int i = t; i < A.nlong; i += BLOCK) v0 += A.part_long[i];
        } else if (lo) {
            // (a word past the end of its list is read from whatever
            // follows and dropped)
            double e[T + 4];
            const u64 *const p = Dk + t, *const pf = Dk + max(far, 0);
            px_poll<T + 4>([&](int i) { return i < T ? p + i * BLOCK : i == T ? p + oCG : pf + (i - T - 1); },
                           [&](int i) { return i < T ? t + i * BLOCK < A.ntile : i == T ? t < A.ncd : far >= 0; }, e, A.ctl, &S.gone[0]);
            if (far >= 0) st3(S.wv, tid, {e[T + 1], e[T + 2], e[T + 3]});
            double f[4] = {0, 0, 0, 0};
#pragma unroll
            for (int u = 0; u < T; ++u) f[u] = e[u];
            v0 = (f[0] + f[1]) + (f[2] + f[3]);
            v0 += e[T];
            for (int i = t + BLOCK; i < A.ncd; i += BLOCK) v0 += px_poll1(Dk + oCG + i, A.ctl, &S.gone[0]);
        } else {
            double e[2 * T + 1];
            const u64 *const p = Dk + t;
            px_poll<2 * T + 1>([&](int i) { return i < T ? p + oZW + i * BLOCK : i < 2 * T ? p + oRR + (i - T) * BLOCK : p + oZL; },
                               [&](int i) { return i < 2 * T ? t + (i % T) * BLOCK < A.ntile : t < A.nlong; }, e, A.ctl, &S.gone[0]);
            double f[2][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
            for (int u = 0; u < T; ++u) { f[0][u] = e[u]; f[1][u] = e[T + u]; }
            v0 = (f[0][0] + f[0][1]) + (f[0][2] + f[0][3]);
            v1 = (f[1][0] + f[1][1]) + (f[1][2] + f[1][3]);
            v0 += e[2 * T];
            for (int i = t + BLOCK; i < A.nlong; i += BLOCK) v0 += px_poll1(Dk + oZL + i, A.ctl, &S.gone[0]);
        }
        v0 = wave_sum(v0);
        if (!lo) v1 = wave_sum(v1);
        if (lane == 0) { S.sh[0][wave] = v0; S.sh[1][wave] = v1; }
    }
    __syncthreads();
    if (S.gone[0]) return true;
    const double gam = (S.sh[0][0] + S.sh[0][1]) + (S.sh[0][2] + S.sh[0][3]);
    const double rr = (S.sh[1][4] + S.sh[1][5]) + (S.sh[1][6] + S.sh[1][7]);
    double del = (S.sh[0][4] + S.sh[0][5]) + (S.sh[0][6] + S.sh[0][7]);
    be = 0.0;
    bool go = true;
    if (st.a == 2) {
        st.eta2 = st.eta * st.eta * rr;
        go = rr > 0.0;
    } else if (rr <= st.eta2 || st.it >= A.maxit) {
        go = false;
    } else {
        be = gam / st.gam;
        del -= be * gam / st.al;
    }
    if (go && !(del > 0.0)) { go = false; st.indef = true; }   // not positive definite along p: stop
    al = go ? gam / del : 0.0;
    st.gam = gam; st.al = al;
    st.a = go;
    st.it += go;
    return false;
}

template <int T, bool COARSE>
__global__ void __launch_bounds__(PX_NT) k_pcg_resident(PxArgs A)
{
    extern __shared__ double px_smem[];
    PxLds<T> &S = *reinterpret_cast<PxLds<T> *>(px_smem);
    constexpr int OWN = TILE * T;
    const int tid0 = threadIdx.x;
    const PxPart me = A.wg[blockIdx.x];
    const PxScene Q = A.scene[me.scene];
    {
        const int l0 = A.seg_long[me.scene];
        A.nlong = A.seg_long[me.scene + 1] - l0;
        A.ntile = Q.ntile; A.nb = Q.nb; A.bnode0 = Q.bnode0; A.maxit = Q.maxit;
        A.ndom = COARSE ? Q.ndom : 0; A.ncd = CG_SPLIT * A.ndom;
        A.D += 3 * (size_t)px_dlen(Q.tile0, l0, COARSE ? CG_SPLIT * Q.dom0 : 0, Q.body0);
        A.part += Q.tile0; A.part_rr += Q.tile0; A.part_zw += Q.tile0; A.part_long += l0; A.long_rows += l0;
        A.st += 4 * (size_t)me.scene; A.act += me.scene; A.iters += me.scene; A.scal += (size_t)me.scene * NSLOT;
        if (COARSE) {
            A.cg_part += CG_SPLIT * Q.dom0; A.ph_ptr += Q.dom0; A.RC += (size_t)CG_N * Q.dom0;
            A.inv += (size_t)Q.dom0 * CG_N * CG_N;
        }
    }
    const bool tiles = me.tile >= 0;            // a workgroup of tiles, else one of long rows
    const int b = me.tile;
    const int n0 = tiles ? Q.node0 + b * OWN : 0, nend = Q.node0 + TILE * Q.ntile;   // own nodes from n0, before the scene's end
    const int lt0 = b * T;                      // the first own tile among the scene's
    const int dom = b / CG_SPLIT, sl = b % CG_SPLIT;
    const bool cg = COARSE && tiles && dom < A.ndom;
    const int DL = px_dlen(A.ntile, A.nlong, A.ncd, A.nb);
    const int oRR = A.ntile, oZW = 2 * A.ntile, oZL = 3 * A.ntile, oCG = oZL + A.nlong, oWL = oCG + A.ncd, oWB = oWL + 3 * A.nlong;

    int tid = tid0, lane = tid & (TILE - 1), wave = tid / TILE;
    // ---- set-up ---------------------------------------------------------------
    if (tid < 3) S.zs[3 * (OWN + PX_HALO) + tid] = 0.0;
    if (tid < 3) S.res[3 * PX_CHUNK + tid] = 0.0;   // (past rcb)
    static_assert(3 * PX_CHUNK >= CG_N * PX_VROWS, "the zero stays");
    if (tid == 0) { S.nhalo = 0; S.nextra = 0; S.nbody = 0; S.nv = 0; S.fit = 0; S.gone[0] = S.gone[1] = S.gone[2] = S.gone[3] = 0; }
    for (int i = tid; i < PX_HASH; i += PX_NT) S.h.key[i] = -1;
    __syncthreads();
    // the own nodes (threads 0 .. OWN - 1): n
    const int n = n0 + tid;
    const bool own = tiles && tid < OWN && n < nend;
    const int kd0 = own ? A.kind[n] : 2;
    const bool bod = kd0 == 1;
    int ph = -1;          // COARSE: the body translation node that this padding slot stands for
    if (COARSE && cg && tid < OWN)
        for (int u = A.ph_ptr[dom]; u < A.ph_ptr[dom + 1]; ++u)
            if (A.ph_e[u] == sl * OWN + tid) ph = A.ph_n[u];
    if (tid < OWN) {
        const int src = kd0 != 2 ? n : ph;
        S.kind[tid] = kd0 == 2 && ph >= 0 ? 3 : kd0;
        S.bslot[tid] = 0;
        st3(S.px, 2 * OWN + tid, src >= 0 ? ld3(A.r0, src) : d3{0, 0, 0});
        st3(S.px, 3 * OWN + tid, {0, 0, 0});
        st3(S.wv, tid, src >= 0 ? ld3(A.w0, src) : d3{0, 0, 0});
        st3(S.zs, tid, kd0 != 2 ? ld3(A.z0, n) : d3{0, 0, 0});
        S.lidx[tid] = ph >= 0 ? oWB + 3 * ((ph - A.bnode0) / 4) : -1;
        S.vof[tid] = -1;
    }
    __syncthreads();
    if (tid < OWN) {
        st3(S.px, tid, {0, 0, 0});
        st3(S.px, OWN + tid, {0, 0, 0});
    }
    if (bod) {
        // a body's 4 nodes are 4 lanes of one wavefront; the first takes the place
        const int a = n & 3;
        int bslot = 0;
        if (a == 0) bslot = atomicAdd(&S.nbody, 1);
        bslot = __shfl(bslot, lane - a);
        if (bslot >= PX_BODIES) S.fit = 2;
        else {
            S.bslot[tid] = (unsigned char)bslot;
            const double *M = A.dinvB + 144 * (size_t)A.node_body[n - a] + 36 * a;
            for (int q = 0; q < 36; ++q) S.body[144 * bslot + 36 * a + q] = M[q];
        }
        if (COARSE && A.node_da[n] >= 0) {
            const int v = atomicAdd(&S.nv, 1);
            if (v >= PX_VROWS) S.fit = 2;
            else {
                S.vof[tid] = (short)v;
                S.vdom[v] = A.node_da[n] / CG_DOM - Q.dom0;
                S.vgrp[v] = A.node_da[n] % CG_DOM;
            }
        }
    }
    for (int i = tid; i < A.nlong; i += PX_NT) {
        const int q = A.long_rows[i] - n0;
        if (tiles && q >= 0 && q < OWN) S.lidx[q] = oWL + 3 * i;
    }
    // the own rows.  A row is 8 sums as in k_spmv<8> (sum s: blocks s, s + 8,
    // ... of the matrix, then of the pair-local blocks), and a lane takes T of
    // them: with T < 4 one of a row in each of its tiles; with T = 4 four of
    // one row, so that a row's sums meet in two exchanges between two lanes
    // instead of three between eight (the cross-lane sums of 4 tiles took more
    // issue slots than the products).  Sums 0, 1, 4, 5 in the even lane, 2, 3,
    // 6, 7 in the odd one: interior rows of the meshes here have 19 blocks, 3
    // in sums 0 to 2.  First collect the columns that other workgroups own.
    constexpr bool TWO = T == 4;
    auto sum_range = [&](int j, int &k0, int &k1, int &d0, int &d1) {   // blocks k0, k0 + 8, ... < k1 of the lane's sum j
        const int r = n0 + (TWO ? tid >> 1 : TILE * j + tid / 8), sub = TWO ? 2 * (tid & 1) + (j & 1) + 4 * (j >> 1) : tid & 7;
        k0 = k1 = d0 = d1 = 0;
        if (!tiles || r >= nend) return;
        k0 = A.row_ptr[r]; k1 = A.row_ptr[r + 1]; d0 = A.dptr[r]; d1 = A.dptr[r + 1];
        if ((k1 - k0) + (d1 - d0) > LONG_ROW) k1 = k0, d1 = d0;
        k0 += sub; d0 += sub;
    };
    for (int j = 0; j < T; ++j) {
        auto insert = [&](int c) {
            if (c >= n0 && c < n0 + OWN) return;
            unsigned h = ((unsigned)c * 2654435761u) >> 21;
            for (int probe = 0; probe < PX_HASH; ++probe, h = (h + 1) & (PX_HASH - 1)) {
                const int was = atomicCAS(&S.h.key[h], -1, c);
                if (was == c) return;
                if (was == -1) {
                    const int q = atomicAdd(&S.nhalo, 1);
                    if (q < PX_HALO) { S.h.slot[h] = (unsigned short)(OWN + q); S.halo[q] = c; }
                    else S.fit = 2;
                    return;
                }
            }
            S.fit = 2;
        };
        int k0, k1, d0, d1;
        sum_range(j, k0, k1, d0, d1);
        for (int k = k0; k < k1; k += 8) insert(A.col[k]);
        for (int k = d0; k < d1; k += 8) insert(A.dcol[k]);
    }
    static_assert(24 * (OWN + PX_HALO + 1) < 65536, "places in zs are 16 bits");
    static_assert(PX_HASH == 2048, "the hash keeps 11 bits");
    __syncthreads();
    // the first two blocks of every sum into registers, the rest into the extra list
    double B[T][2][9];
    int bi[T], ex[T];   // places of the two columns in zs (bytes, 16 bits each); extras: first | count << 16
    {
        auto place = [&](int c) -> int {
            if (c >= n0 && c < n0 + OWN) return 24 * (c - n0);
            unsigned h = ((unsigned)c * 2654435761u) >> 21;
            for (int probe = 0; probe < PX_HASH; ++probe, h = (h + 1) & (PX_HASH - 1)) {
                if (S.h.key[h] == c) return 24 * S.h.slot[h];
                if (S.h.key[h] == -1) break;
            }
            return 0;   // only after an overflow, which has raised S.fit
        };
#pragma unroll
        for (int j = 0; j < T; ++j) {
            int k0, k1, d0, d1;
            sum_range(j, k0, k1, d0, d1);
            bi[j] = ex[j] = 0;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int k = k0 + 8 * u;
                const bool in = k < k1;
                if (in) bi[j] |= place(A.col[k]) << (16 * u);
#pragma unroll
                for (int q = 0; q < 9; ++q) B[j][u][q] = in ? A.val[9 * (size_t)k + q] : 0.0;
            }
            const int ks = k0 + 16, ds = d0;
            const int m = (ks < k1 ? (k1 - ks + 7) / 8 : 0) + (ds < d1 ? (d1 - ds + 7) / 8 : 0);
            if (m > 0) {
                int f = atomicAdd(&S.nextra, m);
                if (f + m > PX_EXTRA) S.fit = 2;
                else {
                    ex[j] = f | m << 16;
                    for (int k = ks; k < k1; k += 8, ++f) { S.esrc[f] = k; S.eidx[f] = (unsigned short)place(A.col[k]); }
                    for (int k = ds; k < d1; k += 8, ++f) { S.esrc[f] = -1 - k; S.eidx[f] = (unsigned short)place(A.dcol[k]); }
                }
            }
        }
    }
    __syncthreads();
    if (own && kd0 != 2)   // over the lookup table, which no one reads any more
        for (int q = 0; q < 9; ++q) S.mi[9 * tid + q] = A.dinv[9 * (size_t)n + q];
    // the extra blocks: this thread's in registers, then those that LDS keeps
    auto extra_at = [&](int e) { const int c = S.esrc[e]; return c >= 0 ? A.val + 9 * (size_t)c : A.dval + 9 * (size_t)(-1 - c); };
    double Bx[9];
    int zx = 0;
#pragma unroll
    for (int q = 0; q < 9; ++q) Bx[q] = 0.0;
    if (!S.fit) {
        if (tid < S.nextra) {
            const double *M = extra_at(tid);
#pragma unroll
            for (int q = 0; q < 9; ++q) Bx[q] = M[q];
            zx = S.eidx[tid];
        }
        for (int i = tid; i < 9 * min(S.nextra - PX_NT, PX_POOL); i += PX_NT) S.pool[i] = extra_at(PX_NT + i / 9)[i % 9];
    }
    __syncthreads();
    if (S.fit) {   // does not fit: everybody leaves
        if (tid == 0) px_abort(A.ctl, S.fit);
        return;
    }

    // ---- iterations -------------------------------------------------------------
    PxState st;
    st.a = A.act[0];
    st.eta = A.st[2];
    // Why a workgroup's threads leave together: each phase has a flag of its
    // own, raised only before the phase's barrier and read only after it, and
    // another barrier lies between the reads and the phase's next polls.  (The
    // long rows' flag is handed on to the scalars' phase, after the rows'
    // barriers and before that phase's.)
    bool gone = false;
    for (int k = 0; tiles && st.a; ++k) {
        // the thread's number anew in every iteration: what is derived from it
        // is then formed where it is used instead of being kept in registers
        // that the blocks need
        tid = tid0;
        asm volatile("" : "+v"(tid));
        lane = tid & (TILE - 1); wave = tid / TILE;
        const int n = n0 + tid, kd = tid < OWN ? S.kind[tid] : 2, far = tid < OWN ? S.lidx[tid] : -1;
        double al, be;
        gone = px_scalars<T>(A, S, st, k, tid, far, al, be);
        if (gone || !st.a) break;
        u64 *Dn = A.D + (size_t)((k + 1) % 3) * DL, *Dr = A.D + (size_t)((k + 2) % 3) * DL;
        u64 *Zk = A.Z + (size_t)(k & 1) * 3 * A.N, *Zr = A.Z + (size_t)((k + 1) & 1) * 3 * A.N;
        u64 *RCk = A.RC + (size_t)(k & 1) * CG_N * A.ndom_all, *RCr = A.RC + (size_t)((k + 1) & 1) * CG_N * A.ndom_all;
        // ---- the update of the own nodes (k_pcg_step) ----
        d3 zv = {0, 0, 0};
        if (tid < OWN) {
            d3 rv = ld3(S.px, 2 * OWN + tid), sv = ld3(S.px, 3 * OWN + tid);
            if (kd != 2) {
                pcg_sr(ld3(S.wv, tid), al, be, sv, rv);
                st3(S.px, 2 * OWN + tid, rv);
                st3(S.px, 3 * OWN + tid, sv);
            }
            if (COARSE && cg) {
                const d3 v = cg_group_sum(kd == 0 || kd == 3 ? rv : d3{0, 0, 0});
                if ((lane & (CG_AGG - 1)) == CG_AGG - 1) {
                    u64 *p = RCk + (size_t)CG_N * dom + CG_ROWS * sl + 3 * (tid / CG_AGG);
                    px_put(p, v.x); px_put(p + 1, v.y); px_put(p + 2, v.z);
                }
            }
            const d3 zo = ld3(S.zs, tid);
            if (kd == 0) zv = px_mat3v(S.mi + 9 * tid, rv);
            else if (kd == 1) {
                const int q4 = n & 3, first = lane - q4;
                double rb[12];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    rb[3 * q] = __shfl(rv.x, first + q);
                    rb[3 * q + 1] = __shfl(rv.y, first + q);
                    rb[3 * q + 2] = __shfl(rv.z, first + q);
                }
                // the sums of body_rows; one row's words in registers at a time
                const double *M = S.body + 144 * S.bslot[tid] + 36 * q4;
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
            double rz = 0.0, rr = 0.0;
            if (kd < 2) {
                if (!COARSE) {
                    u64 *Zp = Zk + 3 * (size_t)n;
                    px_put(Zp, zv.x); px_put(Zp + 1, zv.y); px_put(Zp + 2, zv.z);
                    st3(S.zs, tid, zv);
                }
                rr = px_dt(rv, rv);
                rz = px_dt(rv, zv);
                d3 pv = ld3(S.px, tid), xv = ld3(S.px, OWN + tid);
                pv = {zo.x + be * pv.x, zo.y + be * pv.y, zo.z + be * pv.z};
                xv = {xv.x + al * pv.x, xv.y + al * pv.y, xv.z + al * pv.z};
                st3(S.px, tid, pv);
                st3(S.px, OWN + tid, xv);
            }
            // empty the words written next time
            if (kd < 2)
#pragma unroll
                for (int q = 0; q < 3; ++q) px_st(Zr + 3 * (size_t)n + q, PX_EMPTY);
            if (tid < T && lt0 + tid < A.ntile) {
                const int t = lt0 + tid;
                px_st(Dr + t, PX_EMPTY); px_st(Dr + oRR + t, PX_EMPTY); px_st(Dr + oZW + t, PX_EMPTY);
            }
            if (COARSE) {
                if (cg && tid == T) px_st(Dr + oCG + CG_SPLIT * dom + sl, PX_EMPTY);
                if (cg && tid >= TILE && tid < TILE + CG_ROWS) px_st(RCr + (size_t)CG_N * dom + CG_ROWS * sl + tid - TILE, PX_EMPTY);
                if (kd == 1 && (n & 3) == 0 && far < 0)
#pragma unroll
                    for (int q = 0; q < 3; ++q) px_st(Dr + oWB + 3 * ((n - A.bnode0) / 4) + q, PX_EMPTY);
            }
            rz = wave_sum(rz); rr = wave_sum(rr);
            if (lane == 0 && lt0 + wave < A.ntile) {
                px_put(Dn + lt0 + wave, rz);
                px_put(Dn + oRR + lt0 + wave, rr);
            }
        }
        if (COARSE) {
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
                const double c = px_poll1(RCk + CG_N * (v < 0 ? dom : S.vdom[v]) + i % CG_N, A.ctl, &S.gone[1]);
                if (v < 0) S.rc[i] = c;
                else S.rcb[CG_N * v + i % CG_N] = c;
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
            if (kd < 2) {
                if (cg && kd == 0) zv = {zv.x + S.zl[3 * (tid / CG_AGG)], zv.y + S.zl[3 * (tid / CG_AGG) + 1], zv.z + S.zl[3 * (tid / CG_AGG) + 2]};
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
        for (int i = tid; i < S.nhalo; i += PX_NT) st3(S.zs, OWN + i, px_poll3(Zk, S.halo[i], A.ctl, &S.gone[2]));
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the emptying stores have completed
        __syncthreads();
        if (S.gone[2]) { gone = true; break; }
        {
            auto z_at = [&](int o) -> d3 {
                const double *q = (const double *)((const char *)S.zs + o);
                return {q[0], q[1], q[2]};
            };
            // the blocks in registers; the extra blocks' products by all
            // threads alike (rows in contact have dozens), to be added to
            // their sums in order
            double p[T][3];
#pragma unroll
            for (int j = 0; j < T; ++j) {
                // (opaque: the places' addresses are formed here, not kept)
                asm volatile("" : "+v"(bi[j]), "+v"(ex[j]));
                p[j][0] = p[j][1] = p[j][2] = 0.0;
                px_acc(B[j][0], z_at(bi[j] & 0xffff), p[j][0], p[j][1], p[j][2]);
                px_acc(B[j][1], z_at((unsigned)bi[j] >> 16), p[j][0], p[j][1], p[j][2]);
                if (T > 2 && (j & 1)) asm volatile("" ::: "memory");   // four z in flight: more would not fit the registers
            }
            asm volatile("" : "+v"(zx));
            if (tid < S.nextra) st3(S.res, tid, px_mat3v(Bx, z_at(zx)));
            for (int lo = 0;;) {
                const int hi = min(lo + PX_CHUNK, S.nextra);
                if constexpr (TWO) {
                    // 256 rows in contact: a chunk is two rounds of blocks from memory, whose loads go out
                    // together (260 -> 266 Newton iterations/s on the 200k-tet squeeze; with fewer tiles, which
                    // rarely have a second round, 1-3 % slower)
                    if (lo == 0 && tid < min(PX_POOL, hi - PX_NT)) st3(S.res, PX_NT + tid, px_mat3v(S.pool + 9 * tid, z_at(S.eidx[PX_NT + tid])));
                    const int e0 = max(lo, PX_NT + PX_POOL) + tid, e1 = e0 + PX_NT;
                    if (e0 < hi) {
                        const double *const M0 = extra_at(e0), *const M1 = extra_at(min(e1, hi - 1));
                        double m0[9], m1[9];
#pragma unroll
                        for (int q = 0; q < 9; ++q) { m0[q] = M0[q]; m1[q] = M1[q]; }
                        st3(S.res, e0 - lo, px_mat3v(m0, z_at(S.eidx[e0])));
                        if (e1 < hi) st3(S.res, e1 - lo, px_mat3v(m1, z_at(S.eidx[e1])));
                    }
                } else {
                    for (int e = max(lo, PX_NT) + tid; e < hi; e += PX_NT)
                        st3(S.res, e - lo, px_mat3v(e < PX_NT + PX_POOL ? S.pool + 9 * (e - PX_NT) : extra_at(e), z_at(S.eidx[e])));
                }
                __syncthreads();
#pragma unroll
                for (int j0 = 0; j0 < T; j0 += 2) {
                    constexpr int P = T < 2 ? T : 2;
                    int x0[P], cnt[P], cmax = 0;   // the sums' entries in the chunk
#pragma unroll
                    for (int u = 0; u < P; ++u) {
                        const int f = ex[j0 + u] & 0xffff, l = f + (ex[j0 + u] >> 16);
                        x0[u] = max(f, lo) - lo;
                        cnt[u] = max(min(l, hi) - lo - x0[u], 0);
                        cmax = max(cmax, cnt[u]);
                    }
                    // (a lane that has none left adds the zero, so that no branch
                    // keeps the sums' reads from overlapping)
                    for (int x = 0; __any(x < cmax); x += 2) {
                        d3 r[2][P];
#pragma unroll
                        for (int h = 0; h < 2; ++h)
#pragma unroll
                            for (int u = 0; u < P; ++u) r[h][u] = ld3(S.res, x + h < cnt[u] ? x0[u] + x + h : PX_CHUNK);
#pragma unroll
                        for (int h = 0; h < 2; ++h)
#pragma unroll
                            for (int u = 0; u < P; ++u) { p[j0 + u][0] += r[h][u].x; p[j0 + u][1] += r[h][u].y; p[j0 + u][2] += r[h][u].z; }
                    }
                }
                lo += PX_CHUNK;
                if (lo >= S.nextra) break;
                __syncthreads();   // the chunk's products are read before the next one's are written
            }
            // a row's A z (the tree of lane_sum<8>), its z.Az, and the tile's sum over 8 rows (wave_sum)
            auto finish = [&](int q, bool first, d3 w) -> double {
                if (!first || n0 + q >= nend || S.lidx[q] >= 0) return 0.0;
                st3(S.wv, q, w);
                if (COARSE) {
                    const int r = n0 + q - A.bnode0;
                    if (r >= 0 && (r & 3) == 0 && r / 4 < A.nb) {
                        u64 *o = Dn + oWB + 3 * (r / 4);
                        px_put(o, w.x); px_put(o + 1, w.y); px_put(o + 2, w.z);
                    }
                }
                return px_dt(ld3(S.zs, q), w);
            };
            if constexpr (TWO) {
                double w[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    double u = p[0][q] + p[1][q], v = p[2][q] + p[3][q];
                    u += dpp_d<DPP_XOR1>(u);
                    v += dpp_d<DPP_XOR1>(v);
                    w[q] = u + v;
                }
                const double dot = sum16(finish(tid >> 1, !(tid & 1), {w[0], w[1], w[2]}));
                if ((lane & 15) == 0) S.shd[wave >> 1][4 * (wave & 1) + (lane >> 4)] = dot;
            } else {
#pragma unroll
                for (int j = 0; j < T; ++j)
#pragma unroll
                    for (int q = 0; q < 3; ++q) p[j][q] = lane_sum<8>(p[j][q]);
                double dot[T];
#pragma unroll
                for (int j = 0; j < T; ++j) dot[j] = finish(TILE * j + tid / 8, (tid & 7) == 0, {p[j][0], p[j][1], p[j][2]});
#pragma unroll
                for (int j = 0; j < T; ++j) dot[j] = wave_sum(dot[j]);
#pragma unroll
                for (int j = 0; j < T; ++j)
                    if (lane == 0) S.shd[j][wave] = dot[j];
            }
        }
        __syncthreads();
        if (tid < T && lt0 + tid < A.ntile) {
            double t = S.shd[tid][0];
            for (int q = 1; q < 8; ++q) t += S.shd[tid][q];
            px_put(Dn + oZW + lt0 + tid, t);
        }
    }
    if (!tiles && me.spare < A.nlong) {
        // ---- long rows spare, spare + nsp, ...; the first one's first blocks in registers ----
        const int r0 = A.long_rows[me.spare], e0 = A.row_ptr[r0] + tid, e1 = A.row_ptr[r0 + 1], f0 = A.dptr[r0] + tid, f1 = A.dptr[r0 + 1];
        const int c0 = e0 < e1 ? A.col[e0] : r0, c1 = f0 < f1 ? A.dcol[f0] : r0;   // absent ones poll the row's own z
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            B[0][0][q] = e0 < e1 ? A.val[9 * (size_t)e0 + q] : 0.0;
            B[0][1][q] = f0 < f1 ? A.dval[9 * (size_t)f0 + q] : 0.0;
        }
        for (int k = 0; st.a; ++k) {
            double al, be;
            gone = px_scalars<T>(A, S, st, k, tid, -1, al, be);
            if (gone || !st.a) break;
            u64 *Dn = A.D + (size_t)((k + 1) % 3) * DL, *Dr = A.D + (size_t)((k + 2) % 3) * DL;
            const u64 *z = A.Z + (size_t)(k & 1) * 3 * A.N;
            if (tid == 0) {
                for (int i = me.spare; i < A.nlong; i += me.nsp) {
                    px_st(Dr + oZL + i, PX_EMPTY);
                    for (int q = 0; q < 3; ++q) px_st(Dr + oWL + 3 * i + q, PX_EMPTY);
                    const int r = A.long_rows[i] - A.bnode0;
                    if (COARSE && r >= 0 && (r & 3) == 0 && r / 4 < A.nb)
                        for (int q = 0; q < 3; ++q) px_st(Dr + oWB + 3 * (r / 4) + q, PX_EMPTY);
                }
            }
            for (int i = me.spare; i < A.nlong; i += me.nsp) {
                int r = r0;
                double ax = 0.0, ay = 0.0, az = 0.0;
                d3 zr;
                auto rest = [&](int q, int end, const int *col, const double *val) {
                    for (; q < end; q += PX_NT) px_acc(val + 9 * (size_t)q, px_poll3(z, col[q], A.ctl, &S.gone[3]), ax, ay, az);
                };
                if (i == me.spare) {   // the first blocks' z and the row's own in one poll
                    const u64 *const p = z + 3u * (unsigned)c0, *const pd = z + 3u * (unsigned)c1, *const pr = z + 3u * (unsigned)r;
                    double v[9];
                    px_poll<9>([&](int i) { return i < 3 ? p + i : i < 6 ? pd + (i - 3) : pr + (i - 6); }, [](int) { return true; }, v, A.ctl, &S.gone[3]);
                    zr = {v[6], v[7], v[8]};
                    if (e0 < e1) px_acc(B[0][0], {v[0], v[1], v[2]}, ax, ay, az);
                    rest(e0 + PX_NT, e1, A.col, A.val);
                    if (f0 < f1) px_acc(B[0][1], {v[3], v[4], v[5]}, ax, ay, az);
                    rest(f0 + PX_NT, f1, A.dcol, A.dval);
                } else {
                    r = A.long_rows[i];
                    zr = px_poll3(z, r, A.ctl, &S.gone[3]);
                    rest(A.row_ptr[r] + tid, A.row_ptr[r + 1], A.col, A.val);
                    rest(A.dptr[r] + tid, A.dptr[r + 1], A.dcol, A.dval);
                }
                ax = wave_sum(ax); ay = wave_sum(ay); az = wave_sum(az);
                if (lane == 0) { S.shl[0][wave] = ax; S.shl[1][wave] = ay; S.shl[2][wave] = az; }
                __syncthreads();
                if (tid == 0) {
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the emptying stores have completed
                    for (int q = 1; q < 8; ++q) { ax += S.shl[0][q]; ay += S.shl[1][q]; az += S.shl[2][q]; }
                    u64 *p = Dn + oWL + 3 * i;
                    px_put(p, ax); px_put(p + 1, ay); px_put(p + 2, az);
                    const int rb = r - A.bnode0;
                    if (COARSE && rb >= 0 && (rb & 3) == 0 && rb / 4 < A.nb) {
                        p = Dn + oWB + 3 * (rb / 4);
                        px_put(p, ax); px_put(p + 1, ay); px_put(p + 2, az);
                    }
                    px_put(Dn + oZL + i, px_dt(zr, {ax, ay, az}));
                }
                __syncthreads();
            }
            if (tid == 0 && S.gone[3]) S.gone[0] = 1;   // the workgroup leaves in the next scalars' phase
        }
    }
    // ---- the end: x, and this workgroup's vote that it has reached it ----
    if (gone) {
        if (tid0 == 0) px_abort(A.ctl, 1);
        return;
    }
    if (own && kd0 != 2) st3(A.x, n, ld3(S.px, OWN + tid0));
    if (tid0 == 0) {
        if (b == 0) {
            A.iters[0] = st.it;
            if (st.indef) A.scal[S_INDEF] = 1.0;
        }
        atomicAdd(A.ctl + 1, 1);
    }
}

// empties the exchange words and clears the control words (abort: the first
// one's value)
__global__ void __launch_bounds__(BLOCK) k_pcgx_fill(int64_t n, u64 *__restrict__ p, int *__restrict__ ctl, int abort)
{
    for (int64_t i = blockIdx.x * (int64_t)BLOCK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLOCK) p[i] = PX_EMPTY;
    if (blockIdx.x == 0 && threadIdx.x < 2) ctl[threadIdx.x] = threadIdx.x == 0 ? abort : 0;
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

template <int T, bool COARSE>
static bool px_allow()
{
    return hipFuncSetAttribute((const void *)k_pcg_resident<T, COARSE>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)sizeof(PxLds<T>)) == hipSuccess;
}

static bool px_coarse(const ipc_ctx *c) { return c->coarse_on && c->n_cdom > 0; }
// a scene's workgroups of T tiles: all its tiles and every slice of its coarse domains
static int px_wgs(const ipc_ctx *c, int s, int T)
{
    const int w = (c->sc[s].nnode_pad / TILE + T - 1) / T;
    return px_coarse(c) ? std::max(w, CG_SPLIT * (c->seg_cdom[s + 1] - c->seg_cdom[s])) : w;
}

// Whether no workgroup of T tiles gets more bodies than it has places for,
// with the coarse correction rows for their groups.  A scene's bodies follow
// each other, 4 nodes each, from bnode0 on.
static bool px_bodies_fit(const ipc_ctx *c, int s, int T)
{
    const SceneInfo &S = c->sc[s];
    const int own = TILE * T, room = (own - (S.bnode0 - S.node0) % own) / 4;   // places in the first workgroup
    const int most = std::max(std::min(S.nb, room), std::min(S.nb - room, own / 4));
    return most <= (px_coarse(c) ? std::min(PX_BODIES, PX_VROWS) : PX_BODIES);
}

// Tiles per workgroup for this context, 0: not for this context.
static int px_tiles(const ipc_ctx *c)
{
    if (c->spmv_lanes != 8 || !c->use_graphs || c->prof || !c->pcg_fused || c->n_long > PX_LONG * c->n_scenes || !c->resident_ok) return 0;
    if (px_coarse(c) && !c->cg_windows) return 0;
    int total = 0, largest[3] = {0, 0, 0};
    const int Ts[3] = {1, 2, 4}, room = c->n_cu - PX_SPARE;   // units for one scene's tiles
    for (int s = 0; s < c->n_scenes; ++s) {
        if (c->sc[s].nnode_pad / TILE > 4 * BLOCK) return 0;
        for (int i = 0; i < 3; ++i) largest[i] = std::max(largest[i], px_wgs(c, s, Ts[i]));
        total += c->sc[s].nnode_pad / TILE;
    }
    for (int i = px_coarse(c) ? 2 : 0; i < 3; ++i)
        if (largest[i] <= std::min(room, BLOCK) && (i == 2 || total + c->n_scenes <= Ts[i] * room)) {
            for (int s = 0; s < c->n_scenes; ++s)
                if (!px_bodies_fit(c, s, Ts[i])) return 0;   // (with more tiles each workgroup has more of them)
            return Ts[i];
        }
    return 0;
}

// The launches of a solve for the scenes on[] (null: all): scenes in order, as
// many as the compute units hold, units left over for long rows, alike for
// each of a launch's scenes.  first: the launches' first workgroups.
//
// At most PX_ROUNDS launches: one after the other each takes its scenes'
// iterations, where the launch-per-iteration form streams all scenes'
// matrices at once (uneven scenes of 1k-40k tets, ms a step, that form and
// this one: 16 scenes, one launch, 48 and 36; 32, two, 44 and 40; 64, four,
// 63 and 71; 256, 13 of them, 236 and 273).
constexpr int PX_ROUNDS = 2;
static bool px_plan(const ipc_ctx *c, int T, const int *on, std::vector<PxPart> &wg, std::vector<int> &first)
{
    const int spare_min = c->n_long > 0 ? 1 : 0;
    for (int s = 0; s < c->n_scenes;) {
        int s1 = s, used = 0, cnt = 0;
        for (; s1 < c->n_scenes; ++s1) {
            if (on && !on[s1]) continue;
            const int w = px_wgs(c, s1, T) + spare_min;
            if (used + w > c->n_cu) break;
            used += w;
            ++cnt;
        }
        if (cnt) {
            if (first.size() == PX_ROUNDS) return false;
            const int most = std::min(c->n_long, c->n_scenes == 1 ? PX_LONG : PX_SPARE);
            const int nsp = spare_min ? std::max(1, std::min(most, 1 + (c->n_cu - used) / cnt)) : 0;
            first.push_back((int)wg.size());
            for (int q = s; q < s1; ++q) {
                if (on && !on[q]) continue;
                const int w = px_wgs(c, q, T);
                for (int k = 0; k < w; ++k) wg.push_back({q, k, 0, 0});
                for (int k = 0; k < nsp; ++k) wg.push_back({q, -1, k, nsp});
            }
        }
        if (s1 == s) return false;   // a scene alone does not fit
        s = s1;
    }
    first.push_back((int)wg.size());
    return true;
}

// exchange words of a context of N nodes and NB bodies
static size_t px_words(int n_scenes, int N, int NB)
{
    const int ndom = N / (CG_AGG * CG_DOM) + n_scenes;
    return 3 * (size_t)px_dlen(N / TILE, PX_LONG * std::min(n_scenes, 64), CG_SPLIT * ndom, NB) + 6 * (size_t)N + 2 * (size_t)CG_N * ndom;
}

size_t pcg_resident_bytes(int n_scenes, int N, int NB)
{
    return Arena::round(8 * px_words(n_scenes, N, NB)) + Arena::round(2 * sizeof(int)) + Arena::round(n_scenes * sizeof(PxScene)) +
           Arena::round(PX_ROUNDS * (size_t)PX_WGMAX * sizeof(PxPart));
}

// The exchange memory of a new context.  A workspace context takes it only
// when the plan's slack stays free for the requests of later calls, so that
// a workspace sized by an earlier plan serves as it did.
void pcg_resident_setup(ipc_ctx *c)
{
    const int ns = c->n_scenes;
    if (c->ws.base) {
        const size_t need = pcg_resident_bytes(ns, c->N, c->NB);
        if (c->ws.used + need + c->ws.size / 17 + (1 << 20) > c->ws.size) return;
    }
    int cu = 0;
    if (hipGetDevice(&c->device) != hipSuccess || hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess)
        return;
    // a stream may be restricted to some of the compute units
    unsigned int mask[64] = {};
    if (hipExtStreamGetCUMask(c->stream, 64, mask) == hipSuccess) {
        int units = 0;
        for (unsigned int m : mask) units += __builtin_popcount(m);
        if (units > 0) cu = std::min(cu, units);
    } else {
        (void)hipGetLastError();
    }
    c->n_cu = std::min(cu, PX_WGMAX);
    if (!px_allow<1, false>() || !px_allow<2, false>() || !px_allow<4, false>() || !px_allow<4, true>()) return;
    // Its sums are those of 8 lanes per row: the PCG's products take 8, unless
    // a count is forced or the scenes take too many launches together (then it
    // serves a Newton iteration's last scenes while the lanes are 8).
    const int lanes = c->spmv_lanes;
    c->spmv_lanes = 8;
    c->resident_ok = true;
    const int T = px_tiles(c);
    c->resident_ok = T > 0;
    std::vector<PxPart> wg;
    std::vector<int> first;
    c->resident_lanes = c->resident_ok && !c->spmv_lanes_forced && px_plan(c, T, nullptr, wg, first);
    c->spmv_lanes = lanes;
    if (!c->resident_ok) return;
    std::vector<int> tab;
    for (int s = 0; s < ns; ++s) {
        const SceneInfo &S = c->sc[s];
        const PxScene q = {S.node0, S.nnode_pad / TILE, S.node0 / TILE, c->seg_cdom[s], c->seg_cdom[s + 1] - c->seg_cdom[s], S.body0, S.nb, S.bnode0, S.max_pcg};
        const int *w = (const int *)&q;
        tab.insert(tab.end(), w, w + sizeof(q) / sizeof(int));
    }
    c->d.px_scene.alloc(tab.size());
    upload_async(c, c->d.px_scene.p, tab.data(), tab.size() * sizeof(int));
    c->d.px_wg.alloc(PX_ROUNDS * (size_t)PX_WGMAX * sizeof(PxPart) / sizeof(int));
    c->d.px_words.alloc(px_words(ns, c->N, c->NB));
    c->d.px_ctl.alloc(2);
}

static std::mutex g_resident_mu[64];   // one resident solve per device at a time

PcgResident pcg_resident(ipc_ctx *c, double *x, const int *on)
{
    const int T = px_tiles(c);
    if (!T) return PCG_RESIDENT_NO;
    Dev &D = c->d;
    if (!D.px_words.p) return PCG_RESIDENT_NO;
    if (c->resident_skip > 0) { --c->resident_skip; return PCG_RESIDENT_NO; }
    // workgroups of two resident launches could each hold compute units the
    // other waits for; the lock is kept until this one's end is known
    std::unique_lock<std::mutex> lock(g_resident_mu[c->device & 63], std::try_to_lock);
    if (!lock.owns_lock()) return PCG_RESIDENT_NO;
    hipStream_t st = c->stream;
    const bool coarse = px_coarse(c);
    std::vector<PxPart> wg;
    std::vector<int> round;
    if (!px_plan(c, T, on, wg, round)) return PCG_RESIDENT_NO;
    const int wgs = (int)wg.size();
    if (wgs == 0 || D.px_wg.n < wgs * sizeof(PxPart) / sizeof(int)) return PCG_RESIDENT_NO;
    PxArgs A{};
    A.N = c->N;
    A.ntile = c->N / TILE; A.nlong = c->n_long; A.nb = c->NB; A.ncd = coarse ? CG_SPLIT * c->n_cdom : 0; A.ndom = A.ndom_all = coarse ? c->n_cdom : 0;
    const int64_t nd = 3 * (int64_t)px_dlen(A.ntile, A.nlong, A.ncd, A.nb), nz = 6 * (int64_t)A.N, nr = 2 * (int64_t)CG_N * A.ndom;
    if ((size_t)(nd + nz + nr) > D.px_words.n) return PCG_RESIDENT_NO;
    A.scene = (const PxScene *)D.px_scene.p; A.wg = (const PxPart *)D.px_wg.p; A.seg_long = seg_ptr(c, R_LONG);
    A.kind = D.node_kind.p; A.node_body = D.node_body.p; A.row_ptr = D.row_ptr.p; A.col = D.col.p; A.dptr = D.dyn_ptr.p; A.dcol = D.dyn_col.p;
    A.long_rows = D.long_rows.p; A.node_da = D.cg_node_da.p;
    A.val = D.val.p; A.dval = D.dyn_val.p; A.dinv = D.dinv.p; A.dinvB = D.dinvB.p; A.inv = D.cg_inv.p;
    A.r0 = D.r.p; A.z0 = D.z.p; A.w0 = D.w.p;
    A.part = D.pcg_part.p; A.part_rr = A.part + A.ntile; A.part_zw = D.part_node3.p; A.part_long = D.part_long.p; A.cg_part = D.cg_part.p;
    A.st = D.pcg_st.p; A.act = D.pcg_act.p;
    A.ph_ptr = D.cg_ph_ptr.p; A.ph_e = D.cg_ph_e.p; A.ph_n = D.cg_ph_n.p;
    A.x = x; A.scal = D.scal.p; A.iters = D.pcg_iters.p; A.ctl = D.px_ctl.p;
    A.D = D.px_words.p; A.Z = A.D + nd; A.RC = A.Z + nz;
    upload_async(c, D.px_wg.p, wg.data(), wgs * sizeof(PxPart));
    hipLaunchKernelGGL(k_pcgx_fill, dim3(std::min(blocks_for(nd + nz + nr), 1024)), dim3(BLOCK), 0, st, nd + nz + nr, A.D, A.ctl,
                       c->resident_give_up ? 1 : 0);
    for (size_t k = 0; k + 1 < round.size(); ++k) {
        const int w = round[k + 1] - round[k];
        A.wg = (const PxPart *)D.px_wg.p + round[k];
        switch (T) {
        case 1: px_launch<1, false>(A, w, st); break;
        case 2: px_launch<2, false>(A, w, st); break;
        default:
            if (coarse) px_launch<4, true>(A, w, st);
            else px_launch<4, false>(A, w, st);
        }
    }
    IPC_HIP(hipGetLastError());
    const unsigned int seq = pcg_next_seq(c);
    hipLaunchKernelGGL(k_pcgx_end, dim3(1), dim3(1), 0, st, wgs, D.px_ctl.p, seq, c->h_peek_dev);
    const int status = pcg_await(c, 0, seq, 1);
    if (status == 1) {
        ++c->resident_solves;
        c->resident_waits = 0;
        return PCG_RESIDENT_DONE;
    }
    // The launch-per-iteration form for a while.  A refused set-up costs little
    // to try again; a wait that ran out has cost PX_WAIT, as much as ten
    // solves, so each that follows another doubles the pause (up to 4096
    // solves: a four-hundredth of the time lost, where 64 would lose a tenth).
    c->resident_skip = status == 3 ? 256 : 64 << std::min(c->resident_waits++, 6);
    return PCG_RESIDENT_FAILED;
}

} // namespace ipc
