// Coarse level of the two-level preconditioner: the trilinear (Q1)
// functions on the interior vertices of the same mesh, solved exactly by
// fast diagonalisation in FP64.
//
// Transfers, per cell K with local nodes (a, b, c) at reference coordinates
// (xi_a, xi_b, xi_c) (the GLL nodes) and 1D hats h0(xi) = 1 - xi,
// h1(xi) = xi:
//   restriction   c_v = sum_K sum_(a,b,c) t_K(a,b,c) h_sx(xi_a) h_sy(xi_b) h_sz(xi_c)
//                 over the cells K having v as corner (sx, sy, sz): the Q1 basis
//                 functions tested against the dual residual, which depends on
//                 t only through its assembly G^T t;
//   prolongation  z_K(a,b,c) += sum_corners e_v h_sx(xi_a) h_sy(xi_b) h_sz(xi_c)
//                 (trilinear interpolation; boundary vertices carry 0).
// The coarse operator of the nested spaces is the Q1 Laplacian of the mesh,
// a Kronecker sum of 1D matrices, so A_0^{-1} = (Sx (x) Sy (x) Sz)
// diag(1/(lx + ly + lz)) (Sx (x) Sy (x) Sz)^T with the 1D generalised
// eigenvectors S (S^T M S = I) of the interior vertices.
#include <algorithm>
#include <mutex>
#include <vector>

#include "fem_internal.h"
#include "host_api.h"
#include "launch.h"
#include "mixed.h"
#include "trace.h"

namespace fem {

// The GLL nodes of each degree, computed once per process.
static const std::vector<double>& gll_cached(int p) {
    static std::once_flag once[kMaxP + 1];
    static std::vector<double> nodes[kMaxP + 1];
    std::call_once(once[p], [p]() { nodes[p] = host_gll_nodes(p); });
    return nodes[p];
}

struct GllNodes {
    double xi[kMaxP + 1];
};

// Operands of every coarse kernel, per problem entry: a = t (dual, the
// storage precision S), c = z (primal, S), d = corner sums
// ([8][nblk * 64] doubles), e = two coarse vectors (2 x (n0-1)(n1-1)(n2-1)
// doubles), fd[0..2] = per direction the coarse S ((n-1) x (n-1)) followed by
// lambda (n-1).  Tiles are one storage block (restriction and prolongation),
// one z-plane or 32 z-columns of coarse values (plane solve), or 256 coarse
// values (pass solve) of one problem.
__device__ __forceinline__ int coarse_m(const ProbEntry& pe, int d) { return pe.n[d] > 1 ? pe.n[d] - 1 : 0; }

// Cell -> its 8 corner sums, one workgroup per storage block, lanes on its 64
// cells (every load is a contiguous run) and the z node planes dealt to the
// four wavefronts, whose sums meet in LDS.  Bound by reading t once: one
// thread per cell left a 24^3 mesh with 216 wavefronts, each walking its 512
// values one plane after the other.  Sums in FP64.
// corner[(sx + 2 sy + 4 sz) * nblk * 64 + e].
constexpr int kRestrictLds = 4 * 8 * kLanes * (int)sizeof(double);

template <int P, typename S, bool MULTI>
__device__ __forceinline__ void restrict_cells_body(const LaunchTable& L, const GllNodes& g, int item, int items,
                                                    char* smem) {
    constexpr int N = P + 1, N2 = N * N, NN = N2 * N;
    const int tile = item;
    if (tile >= L.total_tiles) return;              // uniform over the workgroup
    const ProbEntry& pe = entry<MULTI>(L, tile);
    const int lane = threadIdx.x % kLanes, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kLanes));
    const int e = (tile - pe.tile_begin) * kLanes + lane;
    double out[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) out[i] = 0.0;
    if (e < pe.ncells) {
        const S* v = static_cast<const S*>(pe.a) + (size_t)(e / kLanes) * NN * kLanes + lane;
        for (int c = wv; c < N; c += 4) {
            double ux[2][N];
#pragma unroll
            for (int b = 0; b < N; ++b) {
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int a = 0; a < N; ++a) {
                    const double x = load_as<double>(v + (size_t)(a + N * b + N2 * c) * kLanes);
                    s0 += x * (1.0 - g.xi[a]);
                    s1 += x * g.xi[a];
                }
                ux[0][b] = s0;
                ux[1][b] = s1;
            }
            const double wz[2] = {1.0 - g.xi[c], g.xi[c]};
#pragma unroll
            for (int sx = 0; sx < 2; ++sx) {
                double y0 = 0.0, y1 = 0.0;
#pragma unroll
                for (int b = 0; b < N; ++b) {
                    y0 += ux[sx][b] * (1.0 - g.xi[b]);
                    y1 += ux[sx][b] * g.xi[b];
                }
#pragma unroll
                for (int sz = 0; sz < 2; ++sz) {
                    out[sx + 4 * sz] += y0 * wz[sz];
                    out[sx + 2 + 4 * sz] += y1 * wz[sz];
                }
            }
        }
    }
    double* part = reinterpret_cast<double*>(smem);             // [wavefront][corner][cell]
#pragma unroll
    for (int i = 0; i < 8; ++i) part[(wv * 8 + i) * kLanes + lane] = out[i];
    __syncthreads();
    const int stride = pe.nblk * kLanes;
    double* corner = static_cast<double*>(pe.d);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int i = wv + 4 * h;
        double s = part[i * kLanes + lane];
#pragma unroll
        for (int w = 1; w < 4; ++w) s += part[(w * 8 + i) * kLanes + lane];
        corner[(size_t)i * stride + e] = s;
    }
}

template <int P, typename S, bool MULTI>
__global__ void __launch_bounds__(256) k_restrict_cells(LaunchTable L, GllNodes g) {
    __shared__ __align__(16) char smem[kRestrictLds];
    restrict_cells_body<P, S, MULTI>(L, g, blockIdx.x, gridDim.x, smem);
}

// Coarse right-hand side at interior vertex (vi, vj, vk) from the corner
// sums: its eight cells added in ascending cell order.
__device__ __forceinline__ double vertex_sum(const ProbEntry& pe, int vi, int vj, int vk) {
    const int n0 = pe.n[0], n1 = pe.n[1];
    const int stride = pe.nblk * kLanes;
    const double* corner = static_cast<const double*>(pe.d);
    double s = 0.0;
#pragma unroll
    for (int dz = 0; dz < 2; ++dz)
#pragma unroll
        for (int dy = 0; dy < 2; ++dy)
#pragma unroll
            for (int dx = 0; dx < 2; ++dx) {
                // cell (vi-1+dx, ...) has this vertex as its corner (1-dx, 1-dy, 1-dz)
                const int e = (vi - 1 + dx) + n0 * ((vj - 1 + dy) + n1 * (vk - 1 + dz));
                s += corner[(size_t)((1 - dx) + 2 * (1 - dy) + 4 * (1 - dz)) * stride + e];
            }
    return s;
}

// The coarse solve in three launches where a z-plane of coarse values and the
// bases fit in 64 KB of LDS (kPlaneLds): x and y forward per z-plane
// (reading the corner sums), z forward, scaling and z backward per 32
// columns, y and x backward per z-plane.  The work is a few MFLOP, so the
// time is launches and dependent loads: the nine launches of the pass solve
// with one thread per cell and per value (each sum a chain of loads from L2)
// took 257 us for a whole correction on Q7 24^3 cells in FP32, 103 us on Q4
// 21x13x30 and 44 us on Q2 12^3, these five launches 43, 31 and 22 us.  Every
// sum runs over the same terms in the same order as k_coarse_pass (bitwise
// equal).
constexpr int kPlaneLds = 8192;                     // doubles
constexpr int kPlaneThreads = 512;
constexpr int kColumns = 32;

// Doubles of LDS for meshes of m0 x m1 x m2 interior vertices (long: the squares
// of long edges exceed an int).
static constexpr long plane_lds(long m0, long m1) { return 2 * m0 * m1 + (m0 > m1 ? m0 * m0 : m1 * m1); }
static constexpr long column_lds(long m2) { return m2 * m2 + 2 * m2 * kColumns; }
static_assert(plane_lds(50000, 2) > kPlaneLds && plane_lds(30000, 30000) > kPlaneLds && column_lds(50000) > kPlaneLds,
              "long edges must not pass for short ones");

// out(o, r) = sum_i A(i, o) x(i, r) over a plane in LDS, i ascending; the
// value (i, r) sits at i si + r sr, A row-major [m][m].
__device__ __forceinline__ void plane_pass(const double* A, const double* x, double* out, int m, int rows, int si,
                                           int sr, bool o_fastest, int tid, int nt) {
    for (int id = tid; id < m * rows; id += nt) {
        const int o = o_fastest ? id % m : id / rows, r = o_fastest ? id / m : id % rows;
        const double* xr = x + r * sr;
        double s = 0.0;
#pragma unroll 4
        for (int i = 0; i < m; ++i) s += A[i * m + o] * xr[i * si];
        out[o * si + r * sr] = s;
    }
}

// A basis into LDS, as stored (forward: S^T x) or transposed (backward: S x).
__device__ __forceinline__ void load_basis(const double* S, double* A, int m, bool transpose, int tid, int nt) {
    for (int id = tid; id < m * m; id += nt) {
        if (transpose) A[(id % m) * m + id / m] = S[id];
        else A[id] = S[id];
    }
}

// fwd: vertex sums, x then y forward into the second coarse vector; else
// y then x backward from the second coarse vector into the first.
template <bool MULTI>
__global__ void __launch_bounds__(kPlaneThreads) k_coarse_plane(LaunchTable L, int fwd) {
    extern __shared__ double sm[];
    const int tile = blockIdx.x;
    if (tile >= L.total_tiles) return;
    const ProbEntry& pe = entry<MULTI>(L, tile);
    const int m0 = pe.n[0] - 1, m1 = pe.n[1] - 1, m2 = pe.n[2] - 1, np = m0 * m1;
    const int k = tile - pe.tile_begin, tid = threadIdx.x;
    double* x = sm;
    double* w = sm + np;
    double* A = sm + 2 * np;
    double* cv = static_cast<double*>(pe.e);
    double* half1 = cv + (size_t)np * m2 + (size_t)k * np;
    const double* Sx = static_cast<const double*>(pe.fd[0]);
    const double* Sy = static_cast<const double*>(pe.fd[1]);
    for (int id = tid; id < np; id += kPlaneThreads)
        x[id] = fwd ? vertex_sum(pe, 1 + id % m0, 1 + id / m0, 1 + k) : half1[id];
    if (fwd) load_basis(Sx, A, m0, false, tid, kPlaneThreads);
    else load_basis(Sy, A, m1, true, tid, kPlaneThreads);
    __syncthreads();
    if (fwd) plane_pass(A, x, w, m0, m1, 1, m0, true, tid, kPlaneThreads);
    else plane_pass(A, x, w, m1, m0, m0, 1, false, tid, kPlaneThreads);
    __syncthreads();
    if (fwd) load_basis(Sy, A, m1, false, tid, kPlaneThreads);
    else load_basis(Sx, A, m0, true, tid, kPlaneThreads);
    __syncthreads();
    if (fwd) plane_pass(A, w, half1, m1, m0, m0, 1, false, tid, kPlaneThreads);
    else plane_pass(A, w, cv + (size_t)k * np, m0, m1, 1, m0, true, tid, kPlaneThreads);
}

// z forward, division by lx + ly + lz, z backward of 32 columns of the
// second coarse vector, in place.
template <bool MULTI>
__global__ void __launch_bounds__(256) k_coarse_columns(LaunchTable L) {
    extern __shared__ double sm[];
    const int tile = blockIdx.x;
    if (tile >= L.total_tiles) return;
    const ProbEntry& pe = entry<MULTI>(L, tile);
    const int m0 = pe.n[0] - 1, m1 = pe.n[1] - 1, m2 = pe.n[2] - 1, np = m0 * m1;
    const int tid = threadIdx.x, c = tid % kColumns;
    const int col = (tile - pe.tile_begin) * kColumns + c;
    const bool ok = col < np;
    double* A = sm;
    double* x = sm + m2 * m2;
    double* w = x + m2 * kColumns;
    double* v = static_cast<double*>(pe.e) + (size_t)np * m2 + (ok ? col : 0);
    const double* Sz = static_cast<const double*>(pe.fd[2]);
    load_basis(Sz, A, m2, false, tid, 256);
    for (int k = tid / kColumns; k < m2; k += 256 / kColumns) x[k * kColumns + c] = ok ? v[(size_t)k * np] : 0.0;
    __syncthreads();
    const double* lx = static_cast<const double*>(pe.fd[0]) + (size_t)m0 * m0;
    const double* ly = static_cast<const double*>(pe.fd[1]) + (size_t)m1 * m1;
    const double* lz = Sz + (size_t)m2 * m2;
    const double lxy = ok ? lx[col % m0] + ly[col / m0] : 1.0;
    for (int o = tid / kColumns; o < m2; o += 256 / kColumns) {
        double s = 0.0;
#pragma unroll 4
        for (int i = 0; i < m2; ++i) s += A[i * m2 + o] * x[i * kColumns + c];
        s /= lxy + lz[o];
        w[o * kColumns + c] = s;
    }
    __syncthreads();
    for (int o = tid / kColumns; o < m2; o += 256 / kColumns) {
        double s = 0.0;
#pragma unroll 4
        for (int j = 0; j < m2; ++j) s += A[o * m2 + j] * w[j * kColumns + c];
        if (ok) v[(size_t)o * np] = s;
    }
}

// Corner sums -> coarse right-hand side at the interior vertices (the first
// coarse vector), one thread per vertex.
template <bool MULTI>
__global__ void __launch_bounds__(256) k_restrict_vertices(LaunchTable L) {
    const int tile = blockIdx.x;
    if (tile >= L.total_tiles) return;
    const ProbEntry& pe = entry<MULTI>(L, tile);
    const int m0 = coarse_m(pe, 0), m1 = coarse_m(pe, 1), m2 = coarse_m(pe, 2);
    const long v = (long)(tile - pe.tile_begin) * 256 + threadIdx.x;
    if (v >= (long)m0 * m1 * m2) return;
    static_cast<double*>(pe.e)[v] =
        vertex_sum(pe, 1 + (int)(v % m0), 1 + (int)((v / m0) % m1), 1 + (int)(v / ((long)m0 * m1)));
}

// One 1D pass of the coarse fast-diagonalisation solve along `axis` (0 = x)
// from coarse vector `src` (0 or 1) to the other: forward (fwd = 1)
// out(j) = sum_i S(i, j) x(i) (S^T), backward out(i) = sum_j S(i, j) x(j).
// With `scale` the result is divided by lx + ly + lz (the last forward pass).
template <bool MULTI>
__global__ void __launch_bounds__(256) k_coarse_pass(LaunchTable L, int axis, int fwd, int src_half, int scale) {
    const int tile = blockIdx.x;
    if (tile >= L.total_tiles) return;
    const ProbEntry& pe = entry<MULTI>(L, tile);
    const int m0 = coarse_m(pe, 0), m1 = coarse_m(pe, 1), m2 = coarse_m(pe, 2);
    const long tot = (long)m0 * m1 * m2;
    const long id = (long)(tile - pe.tile_begin) * 256 + threadIdx.x;
    if (id >= tot) return;
    const int i0 = (int)(id % m0), i1 = (int)((id / m0) % m1), i2 = (int)(id / ((long)m0 * m1));
    const int m = axis == 0 ? m0 : axis == 1 ? m1 : m2;
    const int o = axis == 0 ? i0 : axis == 1 ? i1 : i2;
    const long stride = axis == 0 ? 1 : axis == 1 ? m0 : (long)m0 * m1;
    double* cv = static_cast<double*>(pe.e);
    const double* x = cv + (src_half ? tot : 0) + (id - (long)o * stride);
    double* dst = cv + (src_half ? 0 : tot);
    const double* Sd = static_cast<const double*>(pe.fd[axis]);
    double s = 0.0;
    if (fwd) {
        for (int i = 0; i < m; ++i) s += Sd[(size_t)i * m + o] * x[(long)i * stride];
    } else {
        for (int j = 0; j < m; ++j) s += Sd[(size_t)o * m + j] * x[(long)j * stride];
    }
    if (scale) {
        const double* lx = static_cast<const double*>(pe.fd[0]) + (size_t)m0 * m0;
        const double* ly = static_cast<const double*>(pe.fd[1]) + (size_t)m1 * m1;
        const double* lz = static_cast<const double*>(pe.fd[2]) + (size_t)m2 * m2;
        s /= lx[i0] + ly[i1] + lz[i2];
    }
    dst[id] = s;
}

// (1 - xi) e0 + xi e1 at node a of N = P + 1 along one direction; the end
// nodes take their vertex value itself.
template <int P>
__device__ __forceinline__ double between(double e0, double e1, int a, double xi) {
    const double m = (1.0 - xi) * e0 + xi * e1;
    return a == 0 ? e0 : a == P ? e1 : m;
}

// z += P_0 e: trilinear interpolation of the coarse correction (the first
// coarse vector) at the cell nodes, along z, then y, then x.  One workgroup
// per storage block, lanes on its cells, the z node planes dealt to the four
// wavefronts (as the restriction).  A node shared by several cells is an end
// node along the shared directions, so every copy takes the same vertex
// values with the same weights (bitwise continuous).  Bound by reading and
// writing z once.
template <int P, typename S, bool MULTI>
__device__ __forceinline__ void prolong_add_body(const LaunchTable& L, const GllNodes& g, int item, int items) {
    using C = typename Prec<S>::C;
    constexpr int N = P + 1, N2 = N * N, NN = N2 * N;
    const int tile = item;
    if (tile >= L.total_tiles) return;
    const ProbEntry& pe = entry<MULTI>(L, tile);
    const int lane = threadIdx.x % kLanes, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kLanes));
    const int e = (tile - pe.tile_begin) * kLanes + lane;
    if (e >= pe.ncells) return;
    const int n0 = pe.n[0], n1 = pe.n[1], n2 = pe.n[2];
    const int m0 = coarse_m(pe, 0), m1 = coarse_m(pe, 1);
    const int i = e % n0, j = (e / n0) % n1, k = e / (n0 * n1);
    const double* ev = static_cast<const double*>(pe.e);
    double cv[8];
#pragma unroll
    for (int sz = 0; sz < 2; ++sz)
#pragma unroll
        for (int sy = 0; sy < 2; ++sy)
#pragma unroll
            for (int sx = 0; sx < 2; ++sx) {
                const int vi = i + sx, vj = j + sy, vk = k + sz;
                const bool in = vi >= 1 && vi <= n0 - 1 && vj >= 1 && vj <= n1 - 1 && vk >= 1 && vk <= n2 - 1;
                cv[sx + 2 * sy + 4 * sz] = in ? ev[(vi - 1) + (long)m0 * ((vj - 1) + (long)m1 * (vk - 1))] : 0.0;
            }
    S* out = static_cast<S*>(pe.c) + (size_t)(e / kLanes) * NN * kLanes + lane;
    for (int c = wv; c < N; c += 4) {
        double p[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) p[q] = between<P>(cv[q], cv[q + 4], c, g.xi[c]);
        S* row = out + (size_t)c * N2 * kLanes;
#pragma unroll
        for (int b = 0; b < N; ++b) {
            const double l0 = between<P>(p[0], p[2], b, g.xi[b]), l1 = between<P>(p[1], p[3], b, g.xi[b]);
#pragma unroll
            for (int a = 0; a < N; ++a) {
                S* dst = row + (size_t)(a + N * b) * kLanes;
                store_from(dst, (C)(load_as<double>(dst) + between<P>(l0, l1, a, g.xi[a])));
            }
        }
    }
}

template <int P, typename S, bool MULTI>
__global__ void __launch_bounds__(256) k_prolong_add(LaunchTable L, GllNodes g) {
    prolong_add_body<P, S, MULTI>(L, g, blockIdx.x, gridDim.x);
}

template <typename F>
static hipError_t by_prec(int prec, F&& f) {
    switch (prec) {
        case FEM_F64: return f(double{});
        case FEM_F32: return f(float{});
        case FEM_F16: return f(f16_t{});
        default: return f(bf16_t{});
    }
}

static bool has_coarse(const ProbEntry& e) { return e.n[0] > 1 && e.n[1] > 1 && e.n[2] > 1; }

// Tiles of the cell kernels (one storage block each); a problem without
// interior vertices has no coarse space and takes no correction.
static int coarse_cell_tiles(const ProbEntry& e) { return has_coarse(e) ? e.nblk : 0; }

// Fill the tile ranges of `ents` by `tiles` and stage the table.
template <typename F>
static hipError_t coarse_table(LaunchTable& L, ProbEntry* ents, int nprob, TableStager* st, hipStream_t s, F&& tiles) {
    int t = 0;
    for (int i = 0; i < nprob; ++i) {
        ents[i].tile_begin = t;
        ents[i].ntiles = has_coarse(ents[i]) ? tiles(ents[i]) : 0;
        t += ents[i].ntiles;
    }
    L.nprob = nprob;
    L.total_tiles = t;
    return stage_table(L, ents, nprob, st, s);
}

// The coarse solve's tables: plane and column tiles where every problem of
// the launch fits k_coarse_plane and k_coarse_columns, else tiles of 256
// coarse values for the passes.
struct CoarseSolve {
    bool planes = true;
    long lds_plane = 0, lds_column = 0;
    LaunchTable Lp{}, Lc{}, Lv{};
    bool empty() const { return planes ? Lp.total_tiles == 0 : Lv.total_tiles == 0; }
};

static hipError_t coarse_solve_tables(CoarseSolve& cs, ProbEntry* ents, int nprob, TableStager* st, hipStream_t s) {
    for (int i = 0; i < nprob; ++i) {
        if (!has_coarse(ents[i])) continue;
        cs.lds_plane = std::max(cs.lds_plane, plane_lds(ents[i].n[0] - 1, ents[i].n[1] - 1));
        cs.lds_column = std::max(cs.lds_column, column_lds(ents[i].n[2] - 1));
    }
    cs.planes = cs.lds_plane <= kPlaneLds && cs.lds_column <= kPlaneLds;
    if (!cs.planes)
        return coarse_table(cs.Lv, ents, nprob, st, s, [](const ProbEntry& e) {
            return (int)(((long)(e.n[0] - 1) * (e.n[1] - 1) * (e.n[2] - 1) + 255) / 256);
        });
    hipError_t err = coarse_table(cs.Lp, ents, nprob, st, s, [](const ProbEntry& e) { return e.n[2] - 1; });
    if (err != hipSuccess) return err;
    return coarse_table(cs.Lc, ents, nprob, st, s, [](const ProbEntry& e) {
        return ((e.n[0] - 1) * (e.n[1] - 1) + kColumns - 1) / kColumns;
    });
}

// Corner sums -> the coarse correction in the first coarse vector.
template <bool MULTI>
static void launch_coarse_solve(const CoarseSolve& cs, hipStream_t s) {
    if (cs.planes) {
        const int lp = (int)(cs.lds_plane * sizeof(double)), lc = (int)(cs.lds_column * sizeof(double));
        hipLaunchKernelGGL(k_coarse_plane<MULTI>, dim3(cs.Lp.total_tiles), dim3(kPlaneThreads), lp, s, cs.Lp, 1);
        hipLaunchKernelGGL(k_coarse_columns<MULTI>, dim3(cs.Lc.total_tiles), dim3(256), lc, s, cs.Lc);
        hipLaunchKernelGGL(k_coarse_plane<MULTI>, dim3(cs.Lp.total_tiles), dim3(kPlaneThreads), lp, s, cs.Lp, 0);
        return;
    }
    const dim3 grid(cs.Lv.total_tiles), block(256);
    hipLaunchKernelGGL(k_restrict_vertices<MULTI>, grid, block, 0, s, cs.Lv);
    // x, y, z forward (then the eigenvalue scaling), z, y, x backward;
    // vector 0 -> 1 -> 0 -> 1 -> 0 -> 1 -> 0
    const int axis[6] = {0, 1, 2, 2, 1, 0}, fwd[6] = {1, 1, 1, 0, 0, 0};
    for (int k = 0; k < 6; ++k)
        hipLaunchKernelGGL(k_coarse_pass<MULTI>, grid, block, 0, s, cs.Lv, axis[k], fwd[k], k % 2, k == 2 ? 1 : 0);
}

template <int P>
static hipError_t coarse_p(int prec, ProbEntry* ents, int nprob, TableStager* st, hipStream_t s) {
    GllNodes g{};
    const std::vector<double>& xi = gll_cached(P);
    for (int a = 0; a <= P; ++a) g.xi[a] = xi[a];
    LaunchTable Lc{};
    hipError_t err = coarse_table(Lc, ents, nprob, st, s, coarse_cell_tiles);
    if (err != hipSuccess) return err;
    if (Lc.total_tiles == 0) return hipSuccess;     // no interior vertex anywhere: no coarse space
    CoarseSolve cs;
    err = coarse_solve_tables(cs, ents, nprob, st, s);
    if (err != hipSuccess) return err;
    const dim3 grid(Lc.total_tiles), block(256);
    return by_prec(prec, [&](auto tag) {
        using S = decltype(tag);
        TraceSpan ts("coarse_correction", P, Prec<S>::id, s);
        if (nprob > 1) {
            hipLaunchKernelGGL((k_restrict_cells<P, S, true>), grid, block, 0, s, Lc, g);
            launch_coarse_solve<true>(cs, s);
            hipLaunchKernelGGL((k_prolong_add<P, S, true>), grid, block, 0, s, Lc, g);
        } else {
            hipLaunchKernelGGL((k_restrict_cells<P, S, false>), grid, block, 0, s, Lc, g);
            launch_coarse_solve<false>(cs, s);
            hipLaunchKernelGGL((k_prolong_add<P, S, false>), grid, block, 0, s, Lc, g);
        }
        return hipGetLastError();
    });
}

// Mixed-degree coarse correction: restriction and prolongation as mixed
// launches (cell tiles of the degrees 7, 3, 2), the coarse solve (the same for
// every degree) over all problems at once.
template <int P, typename S>
struct RestrictBody {
    using Arg = GllNodes;
    static constexpr int kLds = kRestrictLds;
    __device__ static __forceinline__ void run(const LaunchTable& L, const GllNodes& g, int item, int items, char* smem) {
        restrict_cells_body<P, S, true>(L, g, item, items, smem);
    }
};

template <int P, typename S>
struct ProlongBody {
    using Arg = GllNodes;
    static constexpr int kLds = 0;
    __device__ static __forceinline__ void run(const LaunchTable& L, const GllNodes& g, int item, int items, char*) {
        prolong_add_body<P, S, true>(L, g, item, items);
    }
};

static GllNodes gll_arg(int p) {
    GllNodes g{};
    const std::vector<double>& xi = gll_cached(p);
    for (int a = 0; a <= p; ++a) g.xi[a] = xi[a];
    return g;
}

static hipError_t coarse_mixed(int prec, ProbEntry* ents, int nprob, TableStager* st, hipStream_t s) {
    static_assert(mix_degree(0) == 7 && mix_degree(1) == 3 && mix_degree(2) == 2, "segment degrees");
    CoarseSolve cs;
    hipError_t err = coarse_solve_tables(cs, ents, nprob, st, s);
    if (err != hipSuccess) return err;
    if (cs.empty()) return hipSuccess;              // no interior vertex anywhere: no coarse space
    MixTable T{};
    int grid = 0;
    auto tiles = [](int, const ProbEntry& e) { return coarse_cell_tiles(e); };
    auto items = [](int, int t) { return t; };
    err = mix_build(ents, nprob, st, s, tiles, items, T, grid);
    if (err != hipSuccess) return err;
    const GllNodes g7 = gll_arg(7), g3 = gll_arg(3), g2 = gll_arg(2);
    return by_prec(prec, [&](auto tag) {
        using S = decltype(tag);
        TraceSpan ts("coarse_correction", 0, Prec<S>::id, s);
        if (grid > 0)
            hipLaunchKernelGGL((k_mixed<RestrictBody<7, S>, RestrictBody<3, S>, RestrictBody<2, S>>), dim3(grid),
                               dim3(256), 0, s, T, g7, g3, g2);
        launch_coarse_solve<true>(cs, s);
        if (grid > 0)
            hipLaunchKernelGGL((k_mixed<ProlongBody<7, S>, ProlongBody<3, S>, ProlongBody<2, S>>), dim3(grid),
                               dim3(256), 0, s, T, g7, g3, g2);
        return hipGetLastError();
    });
}

hipError_t launch_coarse_any(int prec, ProbEntry* ents, int nprob, TableStager* st, hipStream_t s, bool mix) {
    if (nprob <= 0) return hipSuccess;
    if (mix && mix_degrees(ents, nprob) >= 2) return coarse_mixed(prec, ents, nprob, st, s);
    std::vector<ProbEntry> g;
    for (int p = 1; p <= kMaxP; ++p) {
        g.clear();
        for (int i = 0; i < nprob; ++i)
            if (ents[i].p == p) g.push_back(ents[i]);
        if (g.empty()) continue;
        hipError_t err = launch_coarse_correction(p, prec, g.data(), (int)g.size(), st, s);
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

// Entry of a problem for the coarse kernels: a = t, c = z.
ProbEntry coarse_entry(fem_problem* P, const void* t, void* z) {
    ProbEntry e = entry_of(P);
    e.a = t;
    e.c = z;
    e.d = P->d_corner;
    e.e = P->d_cvec;
    for (int k = 0; k < 3; ++k) e.fd[k] = P->d_cfd + P->cfd_off[k];
    return e;
}

hipError_t launch_coarse_correction(int p, int prec, ProbEntry* ents, int nprob, TableStager* st, hipStream_t s) {
    if (nprob <= 0) return hipSuccess;
    switch (p) {
        case 1: return coarse_p<1>(prec, ents, nprob, st, s);
        case 2: return coarse_p<2>(prec, ents, nprob, st, s);
        case 3: return coarse_p<3>(prec, ents, nprob, st, s);
        case 4: return coarse_p<4>(prec, ents, nprob, st, s);
        case 5: return coarse_p<5>(prec, ents, nprob, st, s);
        case 6: return coarse_p<6>(prec, ents, nprob, st, s);
        case 7: return coarse_p<7>(prec, ents, nprob, st, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t run_coarse_correction(fem_problem* P, const void* t, void* z, int prec) {
    ProbEntry e = coarse_entry(P, t, z);
    return launch_coarse_correction(P->p, prec, &e, 1, nullptr, P->stream);
}

}  // namespace fem
