// Dual-mesh mapping (Sec. III-D, Eq. (6)-(7)): W = S^(L) ... S^(1), the L-level
// Loop subdivision of the coarse simulation mesh as one sparse matrix, built
// on the host at creation; X^f = W X^c for many frames per launch.
//
// The application is HBM-bound: W is read once per launch and every frame
// writes 24 B per fine vertex, while the coarse frames (24 B per coarse
// vertex) stay in L2.  A thread keeps its rows of W in registers and loops
// over the frames (k_dm_pairs; k_dm_frame where a workgroup has one frame;
// k_dm_rows where W's own rows are the smaller form; k_dm_apply for long
// rows).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <iterator>
#include <memory>
#include <mutex>
#include <stdexcept>
#include <string>
#include <unordered_map>
#include <vector>

#include "../../include/ipc.h"
#include "../../include/ipc_dualmesh.h"

struct ipc_dualmesh {
    hipStream_t stream = nullptr;
    int n_coarse = 0, n_fine = 0, max_row = 0, max_group = 0;   // columns of the widest row, of the widest group
    int64_t nnz = 0;
    std::vector<int> row_ptr, col, tri_fine;
    std::vector<double> val;
    // W for k_dm_pairs (empty if a row has more than DM_K columns): groups of
    // one or two rows (rows of group g: grp_row[g] .. grp_row[g + 1]), blocks
    // of at most DM_T groups, each with the list of its distinct columns
    // (in blk_cols) and, by [k][group of the block], the group's k-th
    // column's place in that list (times 3) and, by [k][row of the group][group], its
    // weights (grp_col, grp_val)
    struct Block {
        int u0, nu;    // its columns: blk_cols[u0 .. u0 + nu)
        int g0, ng;    // its groups
        int w0, nk;    // its part of grp_col from w0 on, of grp_val from 2 w0 on; columns of its widest group
        int pad[2];
    };
    std::vector<int> grp_row, blk_cols;
    std::vector<Block> blk;
    std::vector<uint16_t> grp_col;
    std::vector<double> grp_val;
    // W for k_dm_rows (if the no-alloc path or few frames take it): blocks of DM_T rows, block b with
    // its distinct columns row_cols[row_off[b] .. row_off[b + 1]), and every
    // nonzero's column's place in that list (times 3)
    std::vector<int> row_off, row_cols;
    std::vector<uint16_t> row_place;
    uint64_t id = 0;   // unique per handle: names the W that the no-alloc path last staged
    unsigned char *d_w = nullptr;   // the arrays of W, at layout()'s offsets
    unsigned char *d_rows = nullptr;   // and for few frames, row by row
    std::string err;
    ~ipc_dualmesh()
    {
        if (d_w) (void)hipFree(d_w);
        if (d_rows) (void)hipFree(d_rows);
    }
};

namespace {

std::string g_dm_create_error;

constexpr int DM_T = 256;        // groups of rows per workgroup of k_dm_pairs, at most
constexpr int DM_STAGE = 512;    // coarse vertices a block stages in LDS, at most (12 KiB)
constexpr int DM_ROWSTAGE = 1024;   // the same of k_dm_rows (24 KiB)
constexpr int DM_K = 16;         // columns of a group, at most
constexpr int DM_CUS = 256;

struct Invalid : std::runtime_error {
    using std::runtime_error::runtime_error;
};

struct Csr {
    std::vector<int> ptr{0}, col;
    std::vector<double> val;
    int rows() const { return (int)ptr.size() - 1; }
};

double loop_beta(int n)
{
    const double c = 0.375 + 0.25 * std::cos(2.0 * M_PI / n);
    return (0.625 - c * c) / n;
}

// append one row given as (column, weight) pairs: columns ascending, repeats summed
void push_row(Csr &S, std::vector<std::pair<int, double>> &e)
{
    std::sort(e.begin(), e.end(), [](const std::pair<int, double> &a, const std::pair<int, double> &b) { return a.first < b.first; });
    for (size_t k = 0; k < e.size(); ++k) {
        if (k && e[k].first == S.col.back()) S.val.back() += e[k].second;
        else { S.col.push_back(e[k].first); S.val.push_back(e[k].second); }
    }
    S.ptr.push_back((int)S.col.size());
}

// One level: the subdivision matrix S (old vertices, then one row per edge,
// over the old vertices) and the level's triangles.
void loop_level(int n_old, const std::vector<int> &tri, Csr &S, std::vector<int> &tri_out)
{
    const size_t m = tri.size() / 3;
    std::unordered_map<uint64_t, int> eid;
    eid.reserve(3 * m);
    std::vector<int> ea, eb, o0, o1;
    auto key = [](int u, int w) { return ((uint64_t)std::min(u, w) << 32) | (uint64_t)std::max(u, w); };
    std::vector<int> tri_edge(3 * m);
    for (size_t t = 0; t < m; ++t) {
        const int v[3] = {tri[3 * t], tri[3 * t + 1], tri[3 * t + 2]};
        for (int s = 0; s < 3; ++s) {
            const int u = v[s], w = v[(s + 1) % 3], o = v[(s + 2) % 3];
            auto it = eid.find(key(u, w));
            int e;
            if (it == eid.end()) {
                e = (int)ea.size();
                eid.emplace(key(u, w), e);
                ea.push_back(u); eb.push_back(w); o0.push_back(o); o1.push_back(-1);
            } else {
                e = it->second;
                if (o1[e] >= 0) throw Invalid("an edge is shared by more than two triangles");
                o1[e] = o;
            }
            tri_edge[3 * t + s] = e;
        }
    }
    const int ne = (int)ea.size();
    if ((int64_t)n_old + ne > INT32_MAX) throw Invalid("too many fine vertices");
    std::vector<std::vector<int>> nb(n_old), bn(n_old);
    for (int e = 0; e < ne; ++e) {
        nb[ea[e]].push_back(eb[e]);
        nb[eb[e]].push_back(ea[e]);
        if (o1[e] < 0) { bn[ea[e]].push_back(eb[e]); bn[eb[e]].push_back(ea[e]); }
    }
    S = Csr();
    std::vector<std::pair<int, double>> row;
    for (int i = 0; i < n_old; ++i) {
        row.clear();
        if (bn[i].size() > 2) throw Invalid("a vertex lies on more than two boundary edges");
        if (bn[i].size() == 2) {
            row = {{i, 0.75}, {bn[i][0], 0.125}, {bn[i][1], 0.125}};
        } else if (!nb[i].empty()) {
            const int n = (int)nb[i].size();
            const double beta = loop_beta(n);
            row.push_back({i, 1.0 - n * beta});
            for (int j : nb[i]) row.push_back({j, beta});
        } else {
            row.push_back({i, 1.0});
        }
        push_row(S, row);
    }
    for (int e = 0; e < ne; ++e) {
        row.clear();
        if (o1[e] >= 0) row = {{ea[e], 0.375}, {eb[e], 0.375}, {o0[e], 0.125}, {o1[e], 0.125}};
        else row = {{ea[e], 0.5}, {eb[e], 0.5}};
        push_row(S, row);
    }
    tri_out.resize(12 * m);
    for (size_t t = 0; t < m; ++t) {
        const int a = tri[3 * t], b = tri[3 * t + 1], c = tri[3 * t + 2];
        const int ab = n_old + tri_edge[3 * t], bc = n_old + tri_edge[3 * t + 1], ca = n_old + tri_edge[3 * t + 2];
        const int q[12] = {a, ab, ca, b, bc, ab, c, ca, bc, ab, bc, ca};
        for (int k = 0; k < 12; ++k) tri_out[12 * t + k] = q[k];
    }
}

// C = A B (A: rows over B's rows; B: rows over n_cols columns); columns
// ascending per row
Csr multiply(const Csr &A, const Csr &B, int n_cols)
{
    Csr C;
    std::vector<double> acc(n_cols, 0.0);
    std::vector<char> on(n_cols, 0);
    std::vector<int> touched;
    for (int r = 0; r < A.rows(); ++r) {
        touched.clear();
        for (int k = A.ptr[r]; k < A.ptr[r + 1]; ++k) {
            const int i = A.col[k];
            const double a = A.val[k];
            for (int q = B.ptr[i]; q < B.ptr[i + 1]; ++q) {
                const int j = B.col[q];
                if (!on[j]) { on[j] = 1; touched.push_back(j); }
                acc[j] += a * B.val[q];
            }
        }
        std::sort(touched.begin(), touched.end());
        for (int j : touched) { C.col.push_back(j); C.val.push_back(acc[j]); acc[j] = 0.0; on[j] = 0; }
        if (C.col.size() > (size_t)INT32_MAX) throw Invalid("too many nonzeros");
        C.ptr.push_back((int)C.col.size());
    }
    return C;
}

// A fine vertex's 3 doubles, written with non-temporal stores: the output
// (a gigabyte at 100 frames) is written once and never read back by the
// kernel, so it should not displace the coarse frames and W from the caches
// (measured 448 -> 378 us per launch on the cylinder's render mesh).
__device__ __forceinline__ void st_stream(double *o, double x, double y, double z)
{
    __builtin_nontemporal_store(x, o);
    __builtin_nontemporal_store(y, o + 1);
    __builtin_nontemporal_store(z, o + 2);
}

template <int K>
__global__ void __launch_bounds__(256) k_dm_apply(int nf, int nc, int frames, const int *__restrict__ rp, const int *__restrict__ col,
                                                  const double *__restrict__ val, const double *__restrict__ xc,
                                                  double *__restrict__ xf)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nf) return;
    const int k0 = rp[r], n = rp[r + 1] - k0;
    if constexpr (K > 0) {
        int c[K];
        double w[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool in = k < n;
            c[k] = in ? col[k0 + k] : 0;
            w[k] = in ? val[k0 + k] : 0.0;
        }
        for (int f = 0; f < frames; ++f) {
            const double *x = xc + (size_t)f * nc * 3;
            double ax = 0.0, ay = 0.0, az = 0.0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (k < n) {
                    const double *p = x + 3 * (size_t)c[k];
                    ax += w[k] * p[0];
                    ay += w[k] * p[1];
                    az += w[k] * p[2];
                }
            }
            double *o = xf + ((size_t)f * nf + r) * 3;
            st_stream(o, ax, ay, az);
        }
    } else {
        for (int f = 0; f < frames; ++f) {
            const double *x = xc + (size_t)f * nc * 3;
            double ax = 0.0, ay = 0.0, az = 0.0;
            for (int k = 0; k < n; ++k) {
                const double wk = val[k0 + k];
                const double *p = x + 3 * (size_t)col[k0 + k];
                ax += wk * p[0];
                ay += wk * p[1];
                az += wk * p[2];
            }
            double *o = xf + ((size_t)f * nf + r) * 3;
            st_stream(o, ax, ay, az);
        }
    }
}

// Workgroup b takes a block of up to 256 groups of rows, a group (one or two
// consecutive rows with at most KMAX columns between them) per thread, and
// the frames [per blockIdx.y, per (blockIdx.y + 1)).  Per frame it first
// copies the positions of the block's distinct coarse vertices into LDS (each
// fetched once per block: 512 consecutive fine rows touch ~180 coarse
// vertices), then every thread reads its group's columns once for both rows -
// neighbouring fine vertices lie in one coarse triangle and share nearly all
// of their columns, 12.5 for two rows of 11.2 - and the wavefront's rows,
// which are consecutive, go out through LDS as 16 B per lane and whole lines.
//
// What bounds it: the output (24 B per fine vertex and frame), then LDS
// reads.  422402 fine vertices, 100 frames (1014 MB written): 351 us with a
// row per thread, its own CSR row and 8 B stores 24 B apart; 291 with the
// frames in two parts (1650 blocks on 1280 places left the second round
// nearly empty); 258 with two rows per thread (283 with 8 B stores); stores
// straight from two-row threads, 48 B apart,
// 633-1270; three or four rows per thread 289-305 (registers).  One frame
// (118786 fine vertices): 8.4 us with CSR rows, which each thread reads for
// itself, 5.1 with the weights side by side (4.7 in k_dm_frame).
//
// The sums run over a row's own columns in ascending order; the other row's
// columns add 0 * x, which changes nothing unless x is infinite or NaN: a
// block that stages such a position takes the sums with those terms left out.
template <int KMAX>
__global__ void __launch_bounds__(DM_T) k_dm_pairs(int nf, int nc, int frames, int per, const int *__restrict__ grp_row,
                                                   const ipc_dualmesh::Block *__restrict__ blk,
                                                   const int *__restrict__ blk_cols, const uint16_t *__restrict__ grp_col,
                                                   const double *__restrict__ grp_val, const double *__restrict__ xc,
                                                   double *__restrict__ xf)
{
    typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
    constexpr int PER = DM_STAGE / DM_T;   // staged vertices per thread, at most
    __shared__ double sx[3 * DM_STAGE];
    __shared__ double so[6 * DM_T];
    __shared__ int bad[3];                 // a staged position of frame f is not finite: [f mod 3]
    const int t = threadIdx.x, b = blockIdx.x, lane = t & 63;
    const int f0 = blockIdx.y * per, f1 = min(frames, f0 + per);
    const ipc_dualmesh::Block B = blk[b];
    const int ng = B.ng, nk = B.nk;
    int src[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) src[q] = t + q * DM_T < B.nu ? blk_cols[B.u0 + t + q * DM_T] : -1;
    const bool on = t < ng;
    const int ti = min(t, ng - 1);
    int c[KMAX];
    double w[2][KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        c[k] = 0;
        w[0][k] = w[1][k] = 0.0;
    }
    auto load = [&](int k0, int k1) {      // nothing looks at them before the last loads are out
#pragma unroll
        for (int k = k0; k < k1; ++k) {
            const size_t o = (size_t)B.w0 + (size_t)min(k, nk - 1) * ng + ti;
            const size_t v = 2 * o - ti;
            c[k] = grp_col[o];
            w[0][k] = grp_val[v];
            w[1][k] = grp_val[v + ng];
        }
    };
    load(0, 2);
    if (nk > 2) load(2, 6);
    if (nk > 6) load(6, 10);
    if (nk > 10) load(10, 14);
    if (nk > 14) load(14, KMAX);
    // the next frame's staged positions are loaded into registers while this
    // frame is summed and stored, so the gather's latency overlaps the work
    double pf[PER][3];
    auto fetch = [&](int f) {
        const double *x = xc + (size_t)f * nc * 3;
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (src[q] >= 0) {
                pf[q][0] = x[3 * (size_t)src[q]];
                pf[q][1] = x[3 * (size_t)src[q] + 1];
                pf[q][2] = x[3 * (size_t)src[q] + 2];
            }
    };
    if (f0 < f1) fetch(f0);
    const int r0 = grp_row[B.g0 + ti], r1 = grp_row[B.g0 + ti + 1], rows = on ? r1 - r0 : 0;
    int words = 0;                         // of the wavefront's rows, which start at wr0
    const int wr0 = __builtin_amdgcn_readfirstlane(r0), first = __builtin_amdgcn_readfirstlane(t);
    if (first < ng) words = 3 * (__builtin_amdgcn_readlane(r1, min(63, ng - 1 - first)) - wr0);
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        const bool in = k < nk && on;
        c[k] = in ? c[k] : 0;
        w[0][k] = in ? w[0][k] : 0.0;
        w[1][k] = in ? w[1][k] : 0.0;
    }
    int wide = 0;                          // columns of the wavefront's widest group
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
        if (__any(w[0][k] != 0.0 || w[1][k] != 0.0)) wide = k + 1;
    if (t < 3) bad[t] = 0;
    for (int f = f0, slot = 0; f < f1; ++f, slot = slot == 2 ? 0 : slot + 1) {
        __syncthreads();   // the previous frame's reads of sx are done
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (src[q] >= 0) {
                const int u = 3 * (t + q * DM_T);
                sx[u] = pf[q][0];
                sx[u + 1] = pf[q][1];
                sx[u + 2] = pf[q][2];
                if (!(pf[q][0] * 0.0 + pf[q][1] * 0.0 + pf[q][2] * 0.0 == 0.0)) bad[slot] = 1;
            }
        __syncthreads();
        if (t == 0) bad[slot == 0 ? 2 : slot - 1] = 0;   // the previous frame's: read before the barrier above, next set two frames on
        if (f + 1 < f1) fetch(f + 1);
        double a[2][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
        if (!bad[slot]) {
            auto sum = [&](int k0, int k1) {
#pragma unroll
                for (int k = k0; k < k1; ++k) {
                    const double px = sx[c[k]], py = sx[c[k] + 1], pz = sx[c[k] + 2];
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        a[j][0] += w[j][k] * px;
                        a[j][1] += w[j][k] * py;
                        a[j][2] += w[j][k] * pz;
                    }
                }
            };
            sum(0, 6);
            if (wide > 6) sum(6, 10);
            if (wide > 10) sum(10, 14);
            if (wide > 14) sum(14, KMAX);
        } else {
#pragma unroll
            for (int k = 0; k < KMAX; ++k) {
                const double px = sx[c[k]], py = sx[c[k] + 1], pz = sx[c[k] + 2];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const bool in = w[j][k] != 0.0;   // the weights of a row are all positive
                    a[j][0] = in ? __builtin_fma(w[j][k], px, a[j][0]) : a[j][0];
                    a[j][1] = in ? __builtin_fma(w[j][k], py, a[j][1]) : a[j][1];
                    a[j][2] = in ? __builtin_fma(w[j][k], pz, a[j][2]) : a[j][2];
                }
            }
        }
        // the wavefront's own part of so: no barrier
        double *const out = so + 6 * (t - lane);
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (j < rows) {
                double *o = out + 3 * (r0 - wr0 + j);
                o[0] = a[j][0];
                o[1] = a[j][1];
                o[2] = a[j][2];
            }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        double *const o = xf + ((size_t)f * nf + wr0) * 3;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int e = 2 * (64 * q + lane);
            if (e + 1 < words) __builtin_nontemporal_store((d2u){out[e], out[e + 1]}, (d2u *)(o + e));
            else if (e < words) __builtin_nontemporal_store(out[e], o + e);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// One frame per workgroup, for the launches whose frames are split to single
// ones: no loop, no prefetch, and the threads' own sums tell whether a staged
// position is not finite (0 * x is then not 0, and a sum that took one in is
// not finite either; such a thread sums again with the other row's columns
// left out).
//
// What bounds it: three dependent trips to memory, then, with few blocks, the
// loads of one CU: a thread reads up to 48 words of its group.  So NT threads
// take a part of a block's groups, each part staging the block's vertices for
// itself: with 128 threads two CUs share a block as long as there are CUs for
// the halves.  One frame, us, k_dm_pairs / 256 threads / 128: torus of 24 x
// 16, level 1, 3.9 / 3.4 / 3.1; level 2, 4.2 / 3.9 / 3.5; cylinder of 6602
// vertices, level 1 (73 blocks), 4.7 / 4.4 / 3.9, level 3 (885 blocks) 12.4 /
// 12.0 / 12.4.
template <int KMAX, int NT>
__global__ void __launch_bounds__(NT) k_dm_frame(int nf, int nc, const int *__restrict__ grp_row,
                                                 const ipc_dualmesh::Block *__restrict__ blk, const int *__restrict__ blk_cols,
                                                 const uint16_t *__restrict__ grp_col, const double *__restrict__ grp_val,
                                                 const double *__restrict__ xc, double *__restrict__ xf)
{
    typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
    constexpr int PER = DM_STAGE / NT;     // staged vertices per thread, at most
    __shared__ double sx[3 * DM_STAGE];
    __shared__ double so[6 * NT];
    const int tid = threadIdx.x, t = tid + NT * blockIdx.z, lane = tid & 63;
    const size_t f = blockIdx.y;
    const ipc_dualmesh::Block B = blk[blockIdx.x];
    const int ng = B.ng, nk = B.nk;
    if (NT * blockIdx.z >= ng) return;
    int src[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) src[q] = tid + q * NT < B.nu ? blk_cols[B.u0 + tid + q * NT] : -1;
    const bool on = t < ng;
    const int ti = min(t, ng - 1);
    const int r0 = grp_row[B.g0 + ti], r1 = grp_row[B.g0 + ti + 1], rows = on ? r1 - r0 : 0;
    int c[KMAX];
    double w[2][KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        c[k] = 0;
        w[0][k] = w[1][k] = 0.0;
    }
    auto load = [&](int k0, int k1) {      // nothing looks at them before the last loads are out
#pragma unroll
        for (int k = k0; k < k1; ++k) {
            const size_t o = (size_t)B.w0 + (size_t)min(k, nk - 1) * ng + ti;
            const size_t v = 2 * o - ti;
            c[k] = grp_col[o];
            w[0][k] = grp_val[v];
            w[1][k] = grp_val[v + ng];
        }
    };
    load(0, 2);
    if (nk > 2) load(2, 6);
    if (nk > 6) load(6, KMAX < 10 ? KMAX : 10);
    if (KMAX > 10 && nk > 10) load(10, 14);
    if (KMAX > 14 && nk > 14) load(14, KMAX);
    const double *const x = xc + f * nc * 3;
    double px[PER][3];
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (src[q] >= 0)
            for (int m = 0; m < 3; ++m) px[q][m] = x[3 * (size_t)src[q] + m];
    int words = 0;                         // of the wavefront's rows, which start at wr0
    const int wr0 = __builtin_amdgcn_readfirstlane(r0), first = __builtin_amdgcn_readfirstlane(t);
    if (first < ng) words = 3 * (__builtin_amdgcn_readlane(r1, min(63, ng - 1 - first)) - wr0);
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (src[q] >= 0)
            for (int m = 0; m < 3; ++m) sx[3 * (tid + q * NT) + m] = px[q][m];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        const bool in = k < nk && on;
        c[k] = in ? c[k] : 0;
        w[0][k] = in ? w[0][k] : 0.0;
        w[1][k] = in ? w[1][k] : 0.0;
    }
    __syncthreads();
    double a[2][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
    auto sum = [&](int k0, int k1) {
#pragma unroll
        for (int k = k0; k < k1; ++k) {
            const double qx = sx[c[k]], qy = sx[c[k] + 1], qz = sx[c[k] + 2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                a[j][0] += w[j][k] * qx;
                a[j][1] += w[j][k] * qy;
                a[j][2] += w[j][k] * qz;
            }
        }
    };
    sum(0, 2);
    if (nk > 2) sum(2, 6);
    if (nk > 6) sum(6, KMAX < 10 ? KMAX : 10);
    if (KMAX > 10 && nk > 10) sum(10, 14);
    if (KMAX > 14 && nk > 14) sum(14, KMAX);
    const double z = (a[0][0] * 0.0 + a[0][1] * 0.0 + a[0][2] * 0.0) + (a[1][0] * 0.0 + a[1][1] * 0.0 + a[1][2] * 0.0);
    if (!(z == 0.0)) {
#pragma unroll
        for (int j = 0; j < 2; ++j) a[j][0] = a[j][1] = a[j][2] = 0.0;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            const double qx = sx[c[k]], qy = sx[c[k] + 1], qz = sx[c[k] + 2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const bool in = w[j][k] != 0.0;   // the weights of a row are all positive
                a[j][0] = in ? __builtin_fma(w[j][k], qx, a[j][0]) : a[j][0];
                a[j][1] = in ? __builtin_fma(w[j][k], qy, a[j][1]) : a[j][1];
                a[j][2] = in ? __builtin_fma(w[j][k], qz, a[j][2]) : a[j][2];
            }
        }
    }
    // the wavefront's own part of so: no barrier
    double *const out = so + 6 * (tid - lane);
#pragma unroll
    for (int j = 0; j < 2; ++j)
        if (j < rows) {
            double *o = out + 3 * (r0 - wr0 + j);
            o[0] = a[j][0];
            o[1] = a[j][1];
            o[2] = a[j][2];
        }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    double *const o = xf + (f * nf + wr0) * 3;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int e = 2 * (64 * q + lane);
        if (e + 1 < words) __builtin_nontemporal_store((d2u){out[e], out[e + 1]}, (d2u *)(o + e));
        else if (e < words) __builtin_nontemporal_store(out[e], o + e);
    }
}

// Workgroup b takes rows [DM_T b, DM_T b + DM_T), a row per thread from W's
// own rows, and the frames of its part, staging positions as k_dm_pairs does.
// For a W whose pairs, padded to a block's widest group, do not fit the
// no-alloc path's array while its rows do (rows of one or two levels share
// fewer columns).  Cylinder of 8706 vertices, two levels, 139266 rows, 20 and
// 100 frames: 45 and 114 us, k_dm_apply 70 and 349; one level, 237602 rows:
// 56 and 259, 70 and 330.
template <int K>
__global__ void __launch_bounds__(DM_T) k_dm_rows(int nf, int nc, int frames, int per, const int *__restrict__ rp,
                                                  const uint16_t *__restrict__ place, const double *__restrict__ val,
                                                  const int *__restrict__ off, const int *__restrict__ cols,
                                                  const double *__restrict__ xc, double *__restrict__ xf)
{
    constexpr int PER = DM_ROWSTAGE / DM_T;   // staged vertices per thread, at most
    __shared__ double sx[3 * DM_ROWSTAGE];
    const int t = threadIdx.x, r = blockIdx.x * DM_T + t, f0 = blockIdx.y * per, f1 = min(frames, f0 + per);
    const int u0 = off[blockIdx.x], U = off[blockIdx.x + 1] - u0;
    int src[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) src[q] = t + q * DM_T < U ? cols[u0 + t + q * DM_T] : -1;
    int c[K];
    double w[K];
    int n = 0;
    if (r < nf) {
        const int k0 = rp[r];
        n = rp[r + 1] - k0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool in = k < n;
            c[k] = in ? place[k0 + k] : 0;
            w[k] = in ? val[k0 + k] : 0.0;
        }
    }
    double pf[PER][3];
    auto fetch = [&](int f) {
        const double *x = xc + (size_t)f * nc * 3;
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (src[q] >= 0) {
                pf[q][0] = x[3 * (size_t)src[q]];
                pf[q][1] = x[3 * (size_t)src[q] + 1];
                pf[q][2] = x[3 * (size_t)src[q] + 2];
            }
    };
    if (f0 < f1) fetch(f0);
    for (int f = f0; f < f1; ++f) {
        if (f > f0) __syncthreads();   // the previous frame's reads of sx are done
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (src[q] >= 0) {
                const int u = 3 * (t + q * DM_T);
                sx[u] = pf[q][0];
                sx[u + 1] = pf[q][1];
                sx[u + 2] = pf[q][2];
            }
        if (f + 1 < f1) fetch(f + 1);
        __syncthreads();
        if (r < nf) {
            double ax = 0.0, ay = 0.0, az = 0.0;
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (k < n) {
                    ax += w[k] * sx[c[k]];
                    ay += w[k] * sx[c[k] + 1];
                    az += w[k] * sx[c[k] + 2];
                }
            st_stream(xf + ((size_t)f * nf + r) * 3, ax, ay, az);
        }
    }
}

// Groups and blocks of k_dm_pairs (host side of its layout); none for rows of
// more than DM_K columns, nor if the padded groups would not fit the kernel's
// indices (W's own rows do: they go row by row then).
void group_rows(ipc_dualmesh *m)
{
    if (m->max_row > DM_K) return;
    const int kmax = m->max_row > 14 ? 16 : 14, n = m->n_fine;
    const int *rp = m->row_ptr.data(), *col = m->col.data();
    std::vector<int> place(m->n_coarse, -1), cols;      // of the block being filled
    std::vector<int> ucol, uptr{0};                     // each group's columns, ascending
    int g0 = 0, nk = 1;
    bool fits = true;
    auto close = [&](int g1) {
        std::sort(cols.begin(), cols.end());
        for (size_t u = 0; u < cols.size(); ++u) place[cols[u]] = (int)u;
        m->blk_cols.insert(m->blk_cols.end(), cols.begin(), cols.end());
        const int ng = g1 - g0;
        const size_t w0 = m->grp_col.size(), size = w0 + (size_t)nk * ng;
        if (size > (size_t)INT32_MAX) { fits = false; return; }
        m->grp_col.resize(size, 0);
        m->grp_val.resize(2 * size, 0.0);
        for (int g = g0; g < g1; ++g) {
            const int *u = ucol.data() + uptr[g], nu = uptr[g + 1] - uptr[g];
            for (int k = 0; k < nu; ++k) m->grp_col[w0 + (size_t)k * ng + g - g0] = (uint16_t)(3 * place[u[k]]);
            for (int r = m->grp_row[g]; r < m->grp_row[g + 1]; ++r)
                for (int q = rp[r], k = 0; q < rp[r + 1]; ++q) {
                    while (u[k] != col[q]) ++k;
                    m->grp_val[2 * (w0 + (size_t)k * ng) + (size_t)(r - m->grp_row[g]) * ng + g - g0] = m->val[q];
                }
        }
        for (int j : cols) place[j] = -1;
        m->blk.push_back({(int)(m->blk_cols.size() - cols.size()), (int)cols.size(), g0, ng, (int)w0, nk, {0, 0}});
        cols.clear();
        g0 = g1;
        nk = 1;
    };
    m->grp_row.push_back(0);
    for (int r = 0; r < n && fits;) {
        std::vector<int> u;
        int end = r + 1;
        if (end < n) std::set_union(col + rp[r], col + rp[r + 1], col + rp[r + 1], col + rp[r + 2], std::back_inserter(u));
        if (end < n && (int)u.size() <= kmax) ++end;
        else u.assign(col + rp[r], col + rp[r + 1]);
        const int g = (int)m->grp_row.size() - 1;
        int fresh = 0;
        for (int j : u) fresh += place[j] < 0;
        if (g - g0 == DM_T || (int)cols.size() + fresh > DM_STAGE) close(g);
        for (int j : u)
            if (place[j] < 0) { place[j] = 0; cols.push_back(j); }
        nk = std::max(nk, (int)u.size());
        m->max_group = std::max(m->max_group, nk);
        ucol.insert(ucol.end(), u.begin(), u.end());
        uptr.push_back((int)ucol.size());
        m->grp_row.push_back(end);
        r = end;
    }
    if (fits) close((int)m->grp_row.size() - 1);
    if (!fits) {
        m->grp_row.clear(); m->blk_cols.clear(); m->blk.clear(); m->grp_col.clear(); m->grp_val.clear();
        m->max_group = 0;
    }
}

// Blocks of k_dm_rows; none if a block has too many columns.
void list_rows(ipc_dualmesh *m)
{
    if (m->max_row > DM_K) return;
    const int *rp = m->row_ptr.data(), n = m->n_fine;
    std::vector<int> at(m->n_coarse, -1), cols;
    m->row_place.resize(m->col.size());
    m->row_off.push_back(0);
    for (int b0 = 0; b0 < n; b0 += DM_T) {
        const int k0 = rp[b0], k1 = rp[std::min(n, b0 + DM_T)];
        cols.assign(m->col.begin() + k0, m->col.begin() + k1);
        std::sort(cols.begin(), cols.end());
        cols.erase(std::unique(cols.begin(), cols.end()), cols.end());
        if ((int)cols.size() > DM_ROWSTAGE) { m->row_off.clear(); m->row_cols.clear(); m->row_place.clear(); return; }
        for (size_t u = 0; u < cols.size(); ++u) at[cols[u]] = (int)u;
        for (int k = k0; k < k1; ++k) m->row_place[k] = (uint16_t)(3 * at[m->col[k]]);
        m->row_cols.insert(m->row_cols.end(), cols.begin(), cols.end());
        m->row_off.push_back((int)m->row_cols.size());
    }
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// byte offsets of W's arrays on the device, for the kernel of its form; the total
enum Form { PAIRS, ROWS, CSR };   // k_dm_pairs and k_dm_frame; k_dm_rows; k_dm_apply
struct Layout {
    Form form = CSR;
    size_t row = 0, col = 0, val = 0, blk = 0, cols = 0, total = 0;
};
Layout layout(const ipc_dualmesh *m, Form form)
{
    Layout L;
    auto put = [&](size_t bytes) { const size_t o = L.total; L.total += align256(std::max<size_t>(bytes, 1)); return o; };
    L.form = form;
    L.row = put(sizeof(int) * (form == PAIRS ? m->grp_row : m->row_ptr).size());
    L.val = put(sizeof(double) * (form == PAIRS ? m->grp_val : m->val).size());
    L.col = put(form == PAIRS ? sizeof(uint16_t) * m->grp_col.size() : form == ROWS ? sizeof(uint16_t) * m->row_place.size() : sizeof(int) * m->col.size());
    if (form != CSR) {
        L.blk = put(form == PAIRS ? sizeof(ipc_dualmesh::Block) * m->blk.size() : sizeof(int) * m->row_off.size());
        L.cols = put(sizeof(int) * (form == PAIRS ? m->blk_cols : m->row_cols).size());
    }
    return L;
}

hipError_t copy_in(const ipc_dualmesh *m, const Layout &L, unsigned char *base)
{
    hipError_t e = hipSuccess;
    auto put = [&](size_t off, const auto &v) {
        if (e == hipSuccess && !v.empty()) e = hipMemcpyAsync(base + off, v.data(), sizeof(v[0]) * v.size(), hipMemcpyHostToDevice, m->stream);
    };
    switch (L.form) {
    case PAIRS:
        put(L.row, m->grp_row); put(L.val, m->grp_val); put(L.col, m->grp_col);
        put(L.blk, m->blk); put(L.cols, m->blk_cols);
        break;
    case ROWS:
        put(L.row, m->row_ptr); put(L.val, m->val); put(L.col, m->row_place);
        put(L.blk, m->row_off); put(L.cols, m->row_cols);
        break;
    case CSR:
        put(L.row, m->row_ptr); put(L.val, m->val); put(L.col, m->col);
    }
    return e;
}

Layout owned(const ipc_dualmesh *m) { return layout(m, !m->grp_row.empty() ? PAIRS : !m->row_off.empty() ? ROWS : CSR); }

// Whether a few frames (DM_FEW at most) go row by row: what they cost is to
// read W, and where rows are short, of one level, pairs share few columns and
// padded to a block's widest group are the larger form.  Rows of 4.75 columns,
// 1, 2, 4, 8 and 20 frames, by pairs and by rows, us: torus, 240000 rows (712
// blocks), 6.4 / 8.3 / 12.9 / 20.7 / 44 and 5.5 / 7.1 / 11.8 / 20.5 / 46;
// cylinder, 237602 (837), 8.3 / 11.0 / 15.6 / 24.5 / 51 and 5.9 / 8.3 / 13.9 /
// 23.8 / 55; torus, 1200000 (3560, more than run in two rounds), 23.3 / 33.7 /
// 53 / 94 and 22.6 / 34.1 / 56 / 100; with fewer than two blocks per CU
// latency decides (73 blocks: 4.0 and 3.8, 107: 3.7 and 3.8).  Two levels (8.7
// columns, 357 blocks) 6.0 and 6.0, three (11.2) 12.1 and 19.0; none (one
// column), 586 blocks, 4.2 and 4.9.
constexpr int DM_FEW = 4;
bool few_by_rows(const ipc_dualmesh *m)
{
    const int nb = (int)m->blk.size();
    return nb >= 2 * DM_CUS && nb <= 8 * DM_CUS && m->nnz > 2 * (int64_t)m->n_fine && m->nnz < 6 * (int64_t)m->n_fine;
}

// W on the device in one form
hipError_t upload(ipc_dualmesh *m, const Layout &L, unsigned char *&dev)
{
    if (dev) return hipSuccess;
    unsigned char *p = nullptr;
    hipError_t e = hipMalloc(&p, L.total);
    if (e == hipSuccess) e = copy_in(m, L, p);
    if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
    if (e == hipSuccess) dev = p;   // only a W that has arrived is taken for one by the next call
    else if (p) (void)hipFree(p);
    return e;
}
bool by_rows(const ipc_dualmesh *m) { return few_by_rows(m) && !m->row_off.empty(); }
// every form that a call may take, with the first one (so that later calls, under capture too, only launch)
hipError_t upload(ipc_dualmesh *m)
{
    hipError_t e = upload(m, owned(m), m->d_w);
    if (e == hipSuccess && by_rows(m)) e = upload(m, layout(m, ROWS), m->d_rows);
    return e;
}

hipError_t launch(ipc_dualmesh *m, const Layout &L, const unsigned char *base, const double *xc, double *xf, int frames)
{
    const int *row = (const int *)(base + L.row);
    const double *val = (const double *)(base + L.val);
    const int R = m->max_row;
    // Frames are split over blocks: as long as all of the blocks run at once
    // (four per CU), to single frames, which then take as long as one; beyond,
    // to about four rounds of blocks, so that the last, partly empty one
    // weighs little, and at least 16 frames each: a block's set-up reads the
    // weights, as many bytes as five frames write.  k_dm_pairs, 885 blocks by
    // 100 frames: one part 304 us, two 270, three 264, four 259, six 255.  13
    // blocks by 20: one part 28 us, twenty 6.
    const int nb = L.form == PAIRS ? (int)m->blk.size() : (m->n_fine + DM_T - 1) / DM_T;
    const int parts = std::max({1, std::min(4 * DM_CUS / nb, frames), std::min((16 * DM_CUS + nb - 1) / nb, frames / 16)});
    const int per = (frames + parts - 1) / parts;
    if (L.form == ROWS) {
        hipLaunchKernelGGL(k_dm_rows<DM_K>, dim3(nb, (frames + per - 1) / per), dim3(DM_T), 0, m->stream, m->n_fine, m->n_coarse, frames, per,
                           row, (const uint16_t *)(base + L.col), val, (const int *)(base + L.blk), (const int *)(base + L.cols), xc, xf);
        return hipGetLastError();
    }
    if (L.form == PAIRS) {
        const auto *blk = (const ipc_dualmesh::Block *)(base + L.blk);
        const int *cols = (const int *)(base + L.cols);
        const uint16_t *col = (const uint16_t *)(base + L.col);
        auto one = [&](auto kern, int nt) {
            hipLaunchKernelGGL(kern, dim3(nb, frames, DM_T / nt), dim3(nt), 0, m->stream, m->n_fine, m->n_coarse, row, blk, cols, col, val, xc, xf);
        };
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(nb, (frames + per - 1) / per), dim3(DM_T), 0, m->stream, m->n_fine, m->n_coarse, frames, per, row, blk,
                               cols, col, val, xc, xf);
        };
        if (per == 1) {   // at most 1024 frames, or one: blocks halved while every half has a CU (52 blocks: 2 frames 4.4 us whole, 4.0 halved, 4 frames 4.5 and 4.7)
            const bool half = (int64_t)2 * nb * frames <= DM_CUS, narrow = m->max_group <= 8;   // (regular meshes of one level: groups of at most 8)
            if (half) narrow ? one(k_dm_frame<8, DM_T / 2>, DM_T / 2) : one(k_dm_frame<16, DM_T / 2>, DM_T / 2);
            else narrow ? one(k_dm_frame<8, DM_T>, DM_T) : one(k_dm_frame<16, DM_T>, DM_T);
        } else if (R <= 14) go(k_dm_pairs<14>);   // 128 registers: four blocks per CU; regular meshes have rows of at most 14
        else go(k_dm_pairs<16>);
        return hipGetLastError();
    }
    const dim3 grid((m->n_fine + 255) / 256), blk(256);
    const int *col = (const int *)(base + L.col);
#define IPC_DM(KK) hipLaunchKernelGGL(k_dm_apply<KK>, grid, blk, 0, m->stream, m->n_fine, m->n_coarse, frames, row, col, val, xc, xf)
    if (R <= 16) IPC_DM(16);
    else if (R <= 32) IPC_DM(32);
    else if (R <= 48) IPC_DM(48);
    else if (R <= 64) IPC_DM(64);
    else IPC_DM(0);
#undef IPC_DM
    return hipGetLastError();
}

// the product from the library's own memory
hipError_t launch_owned(ipc_dualmesh *m, const double *xc, double *xf, int frames)
{
    return frames <= DM_FEW && by_rows(m) ? launch(m, layout(m, ROWS), m->d_rows, xc, xf, frames) : launch(m, owned(m), m->d_w, xc, xf, frames);
}

// ---- the variant that allocates nothing ------------------------------------
// W is staged in a file-scope device array of fixed size instead of memory
// the library allocates.  Every GPU holds its own copy of the array, at its
// own address, taken once per device with hipGetSymbolAddress; the host-side
// name of the array is not a device address and is never passed to a kernel
// or a copy.  The array keeps the W of the last call on that GPU: a call with
// the same handle does not copy it again.
constexpr size_t DM_SCRATCH_BYTES = 16u << 20;
static __device__ __align__(256) unsigned char scratch[DM_SCRATCH_BYTES];
constexpr int DM_MAX_DEVICES = 64;
struct ScratchSlot {
    unsigned char *ptr = nullptr;   // this device's address of the array
    uint64_t holds = 0;             // id of the handle whose W it holds (0: none)
};
std::mutex g_scratch_mu;
ScratchSlot g_scratch[DM_MAX_DEVICES];
uint64_t g_dm_next_id = 1;

// W as the array holds it: for k_dm_pairs if that fits, else in its own rows,
// staged if they can be and that fits
Layout scratch_layout(const ipc_dualmesh *m)
{
    Layout L = owned(m);
    if (L.total <= DM_SCRATCH_BYTES) return L;
    if (!m->row_off.empty() && (L = layout(m, ROWS)).total <= DM_SCRATCH_BYTES) return L;
    return layout(m, CSR);
}

} // namespace

extern "C" int ipc_dualmesh_create(const int32_t *tri_host, int32_t n_tri, int32_t n_vert, int32_t levels, void *hip_stream,
                                   ipc_dualmesh **out)
{
    if (!out) return IPC_E_INVALID;
    *out = nullptr;
    try {
        if (!tri_host || n_tri < 1 || n_vert < 1) throw Invalid("need at least one triangle and one vertex");
        if (levels < 0 || levels > 6) throw Invalid("levels must lie in [0, 6]");
        if ((int64_t)n_tri << (2 * levels) > INT32_MAX / 3) throw Invalid("too many fine triangles");
        std::vector<int> tri(tri_host, tri_host + 3 * (size_t)n_tri);
        for (int t = 0; t < n_tri; ++t) {
            const int a = tri[3 * t], b = tri[3 * t + 1], c = tri[3 * t + 2];
            if (a < 0 || b < 0 || c < 0 || a >= n_vert || b >= n_vert || c >= n_vert) throw Invalid("vertex index out of range");
            if (a == b || b == c || c == a) throw Invalid("a triangle repeats a vertex");
        }
        auto own = std::make_unique<ipc_dualmesh>();
        ipc_dualmesh *m = own.get();
        m->stream = (hipStream_t)hip_stream;
        {
            std::lock_guard<std::mutex> lock(g_scratch_mu);
            m->id = g_dm_next_id++;
        }
        // W = identity, then one level at a time: W <- S W
        Csr W;
        for (int i = 0; i < n_vert; ++i) { W.col.push_back(i); W.val.push_back(1.0); W.ptr.push_back(i + 1); }
        int n = n_vert;
        for (int l = 0; l < levels; ++l) {
            Csr S;
            std::vector<int> tri_next;
            loop_level(n, tri, S, tri_next);
            W = multiply(S, W, n_vert);
            n = S.rows();
            tri.swap(tri_next);
        }
        m->n_coarse = n_vert;
        m->n_fine = n;
        m->row_ptr = std::move(W.ptr);
        m->col = std::move(W.col);
        m->val = std::move(W.val);
        m->nnz = (int64_t)m->col.size();
        for (int r = 0; r < n; ++r) m->max_row = std::max(m->max_row, m->row_ptr[r + 1] - m->row_ptr[r]);
        m->tri_fine = std::move(tri);
        group_rows(m);
        const bool noalloc = owned(m).total > DM_SCRATCH_BYTES && layout(m, CSR).total <= DM_SCRATCH_BYTES;
        if (m->grp_row.empty() || noalloc || few_by_rows(m)) list_rows(m);
        *out = own.release();
        return IPC_OK;
    } catch (const Invalid &e) {
        g_dm_create_error = e.what();
        return IPC_E_INVALID;
    } catch (const std::exception &e) {
        g_dm_create_error = e.what();
        return IPC_E_DEVICE;
    }
}

extern "C" void ipc_dualmesh_destroy(ipc_dualmesh *m) { delete m; }

extern "C" const char *ipc_dualmesh_last_error(const ipc_dualmesh *m) { return m ? m->err.c_str() : g_dm_create_error.c_str(); }

extern "C" int ipc_dualmesh_query(const ipc_dualmesh *m, int what, int64_t *v)
{
    if (!m || !v) return IPC_E_INVALID;
    switch (what) {
    case IPC_DM_NCOARSE: *v = m->n_coarse; return IPC_OK;
    case IPC_DM_NFINE: *v = m->n_fine; return IPC_OK;
    case IPC_DM_NTRI: *v = (int64_t)(m->tri_fine.size() / 3); return IPC_OK;
    case IPC_DM_NNZ: *v = m->nnz; return IPC_OK;
    case IPC_DM_MAXROW: *v = m->max_row; return IPC_OK;
    }
    return IPC_E_INVALID;
}

extern "C" int ipc_dualmesh_fine_tris(const ipc_dualmesh *m, int32_t *tri_host)
{
    if (!m || !tri_host) return IPC_E_INVALID;
    std::copy(m->tri_fine.begin(), m->tri_fine.end(), tri_host);
    return IPC_OK;
}

extern "C" int ipc_dualmesh_weights(const ipc_dualmesh *m, int32_t *row_ptr, int32_t *col, double *val)
{
    if (!m) return IPC_E_INVALID;
    if (row_ptr) std::copy(m->row_ptr.begin(), m->row_ptr.end(), row_ptr);
    if (col) std::copy(m->col.begin(), m->col.end(), col);
    if (val) std::copy(m->val.begin(), m->val.end(), val);
    return IPC_OK;
}

extern "C" int ipc_dualmesh_apply(ipc_dualmesh *m, const double *xc_dev, double *xf_dev, int32_t n_frames)
{
    if (!m) return IPC_E_INVALID;
    if (!xc_dev || !xf_dev || n_frames < 1) { m->err = "need device arrays and at least one frame"; return IPC_E_INVALID; }
    hipError_t e = upload(m);
    if (e == hipSuccess) e = launch_owned(m, xc_dev, xf_dev, n_frames);
    if (e != hipSuccess) { m->err = std::string("HIP: ") + hipGetErrorString(e); return IPC_E_DEVICE; }
    return IPC_OK;
}

extern "C" int ipc_dualmesh_apply_noalloc(ipc_dualmesh *m, const double *xc_dev, double *xf_dev, int32_t n_frames)
{
    if (!m) return IPC_E_INVALID;
    if (!xc_dev || !xf_dev || n_frames < 1) { m->err = "need device arrays and at least one frame"; return IPC_E_INVALID; }
    const Layout L = scratch_layout(m);
    if (L.total > DM_SCRATCH_BYTES) {
        m->err = "W needs " + std::to_string(L.total) + " bytes of staging; the no-alloc path holds at most " +
                 std::to_string(DM_SCRATCH_BYTES);
        return IPC_E_CAPACITY;
    }
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess && (dev < 0 || dev >= DM_MAX_DEVICES)) { m->err = "device ordinal out of range"; return IPC_E_INVALID; }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    ScratchSlot &S = g_scratch[dev];
    if (e == hipSuccess && !S.ptr) e = hipGetSymbolAddress((void **)&S.ptr, HIP_SYMBOL(scratch));   // once per device
    if (e == hipSuccess && S.holds != m->id) {
        S.holds = 0;
        e = copy_in(m, L, S.ptr);
        if (e == hipSuccess) S.holds = m->id;
    }
    if (e == hipSuccess) e = launch(m, L, S.ptr, xc_dev, xf_dev, n_frames);
    if (e != hipSuccess) { m->err = std::string("HIP: ") + hipGetErrorString(e); return IPC_E_DEVICE; }
    return IPC_OK;
}

extern "C" int ipc_dualmesh_time(ipc_dualmesh *m, const double *xc_dev, double *xf_dev, int32_t n_frames, int32_t reps,
                                 double *avg_us, double *bytes)
{
    if (!m) return IPC_E_INVALID;
    if (!xc_dev || !xf_dev || n_frames < 1 || reps < 1 || !avg_us) { m->err = "invalid timing arguments"; return IPC_E_INVALID; }
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t e = upload(m);
    if (e == hipSuccess) e = launch_owned(m, xc_dev, xf_dev, n_frames);   // warm
    if (e == hipSuccess) e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    if (e == hipSuccess) e = hipEventRecord(e0, m->stream);
    for (int k = 0; k < reps && e == hipSuccess; ++k) e = launch_owned(m, xc_dev, xf_dev, n_frames);
    if (e == hipSuccess) e = hipEventRecord(e1, m->stream);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.0f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (e != hipSuccess) { m->err = std::string("HIP: ") + hipGetErrorString(e); return IPC_E_DEVICE; }
    *avg_us = 1e3 * ms / reps;
    if (bytes)
        *bytes = 12.0 * (double)m->nnz + 4.0 * (m->n_fine + 1.0) + 24.0 * (double)n_frames * ((double)m->n_coarse + m->n_fine);
    return IPC_OK;
}
