// Consumers of the auxiliary-grid potentials (Sec. 6.1, Sec. 7.2): quadrature-weighted
// projections of grid functions on a basis, the exchange action W_a = sum_s psi_s v_as of a set
// of vectors, and the adaptively compressed exchange (ACE) vectors.
//
// Every integral is the grid's quadrature: node q of an element-major field carries the weight
// w_q = m_x[i] m_y[j] m_z[k], the lumped GLL mass of its local indices (the same for every
// element of a uniform mesh).  These steps stream their fields once (the projection reads each
// basis function once), so they are bound by HBM bandwidth.  The projection's sums run on the FP64
// matrix instruction; the other contractions are short and stay on the vector units.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdexcept>

#include "dg_kernels.h"

namespace dg {

namespace {

constexpr int PJ_THREADS = 256;
constexpr int PJ_MAXN3 = 512;  // nodes per element (degree <= 7)
// Chunks of a field: by the mesh alone, and added in pairs of pairs, so that an entry's sum does not depend on
// how many are formed with it.  A work-group takes 1, 2 or 4 of them, fewer where the launch has few tiles, and
// adds them itself.  Whole calls, and with about 512 work-groups a launch, each with one chunk of its own size:
// 256 x 8 entries on 512,000 nodes 0.259 ms (0.266), 8 x 8 0.052 (0.052), 300 x 24 0.529 (0.532), 64 x 8 on
// 4,096,000 nodes 0.492 (0.508), 1000 x 4 on 960,000 1.42 (1.56).  Tried: always one chunk a work-group (the
// 8 MB of partial sums of 256 x 8 entries make the first call 0.5 ms longer).
constexpr int PJ_CHUNKS = 512, PJ_GROUP = 4;
constexpr long long PJ_PARTIAL = 1LL << 28;  // doubles of partial sums a launch may take: more go row block by row block

// 16 bytes of a field whose rows start at any multiple of 8
typedef double pj_d2 __attribute__((ext_vector_type(2), aligned(8)));
typedef double pj_d4 __attribute__((ext_vector_type(4)));

// partial[(i * nu + a) * npart + c] = sum over the nodes q of the chunks c g .. c g + g - 1 of w_q f_q phi_i(q) u_a(q),
// for the 16 RT rows i and the 16 vectors a of this work-group (f null: 1), on
// v_mfma_f64_16x16x4: a wave takes 16 nodes at a time, a lane four neighbouring ones of its row of
// phi (lane & 15), so that each row is read in whole 128-byte pieces, and of its vector of u, whose
// products with w f are the other operand; the four matrix steps take the lanes' first, second, third
// and fourth nodes (tried: 32 rows a work-group, four waves per SIMD, two steps in flight: no faster;
// non-temporal reads: 6% slower).  The reads of phi bound it: u is read once for 16 RT rows of phi (once for 8 in a
// vector form of 8 x 8 sums a thread, which read as much of u from L2 as of phi from memory and
// took 280 us, 3.9 TB/s, for 256 rows and 8 vectors of 512,000 nodes; this form
// 235 us, 4.5 TB/s).
// The weight of a node depends only on its local index in the element (the three 1D lumped masses
// of a uniform mesh), staged in LDS per work-group.  Indices within one field are 32-bit (a field
// has < 2^31 nodes).
template <int RT>
__global__ __launch_bounds__(PJ_THREADS) void k_project(const LevelDev<double>* __restrict__ Lp, int n, int ndof,
                                                        int nbasis, const double* __restrict__ phi, int nu,
                                                        const double* __restrict__ u, const double* __restrict__ f,
                                                        int npart, int g, int cnodes, double* __restrict__ partial) {
    __shared__ double red[PJ_THREADS / 64][RT * 256];
    __shared__ double wloc[PJ_MAXN3 + 3];
    const int nti = (nbasis + 16 * RT - 1) / (16 * RT), nta = (nu + 15) / 16;
    const int b = blockIdx.x;
    const int ti = b % nti, ta = (b / nti) % nta, c = b / (nti * nta);
    const int i0 = ti * 16 * RT, a0 = ta * 16;
    const int n3 = n * n * n;
    {
        const LevelDev<double>& L = *Lp;
        for (int l = threadIdx.x; l < n3 + 3; l += PJ_THREADS) {
            const int m = l % n3;
            wloc[l] = L.ax[0].m[m % n] * L.ax[1].m[(m / n) % n] * L.ax[2].m[m / (n * n)];
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, m = lane & 15, kq = lane >> 4;
    const double* __restrict__ prow[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) prow[t] = phi + (long long)min(i0 + 16 * t + m, nbasis - 1) * ndof;
    const double* __restrict__ urow = u + (long long)min(a0 + m, nu - 1) * ndof;
    double one[RT], all[RT];  // sums of the last even chunk, and of the pairs
#pragma unroll
    for (int t = 0; t < RT; ++t) one[t] = all[t] = 0.0;
    const int dl = 64 % n3;
    for (int k = 0; k < g; ++k) {
        pj_d4 acc[RT];
#pragma unroll
        for (int t = 0; t < RT; ++t) acc[t] = pj_d4{0.0, 0.0, 0.0, 0.0};
        const unsigned q0 = (c * g + k) * (unsigned)cnodes, qe = min((long long)ndof, (long long)q0 + cnodes);
        unsigned q = q0 + wv * 16 + 4 * kq;  // the lane's first node
        int l = q % n3;
        for (; q - 4 * kq + 16 <= qe; q += 64) {
            double pv[RT][4], bv[4];
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const pj_d2 v = *reinterpret_cast<const pj_d2*>(prow[t] + q + 2 * h);
                    pv[t][2 * h] = v[0];
                    pv[t][2 * h + 1] = v[1];
                }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const pj_d2 v = *reinterpret_cast<const pj_d2*>(urow + q + 2 * h);
                pj_d2 w = {wloc[l + 2 * h], wloc[l + 2 * h + 1]};
                if (f) w *= *reinterpret_cast<const pj_d2*>(f + q + 2 * h);
                bv[2 * h] = w[0] * v[0];
                bv[2 * h + 1] = w[1] * v[1];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int t = 0; t < RT; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(pv[t][j], bv[j], acc[t], 0, 0, 0);
            l += dl;
            if (l >= n3) l -= n3;
        }
        if (q - 4 * kq < qe) {  // the field's last, incomplete 16 nodes (one wave of the last chunk)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool ok = q + j < qe;
                const unsigned qq = ok ? q + j : 0;
                double w = ok ? wloc[l + j] : 0.0;
                if (f) w *= f[qq];
                const double bw = w * urow[qq];
#pragma unroll
                for (int t = 0; t < RT; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(prow[t][qq], bw, acc[t], 0, 0, 0);
            }
        }
        // accumulator: vector = lane & 15, row = lane / 16 + 4 * register
        if (k) __syncthreads();  // the last chunk's sums are read
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[wv][t * 256 + (kq + 4 * r) * 16 + m] = acc[t][r];
        __syncthreads();
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < PJ_THREADS / 64; ++w) s += red[w][t * 256 + threadIdx.x];
            if (k & 1)
                all[t] += one[t] + s;
            else
                one[t] = s;
        }
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int i = i0 + 16 * t + (threadIdx.x >> 4), a = a0 + (threadIdx.x & 15);
        if (i < nbasis && a < nu)
            partial[((long long)i * nu + a) * npart + c] = g == 1 ? one[t] : all[t];
    }
}

// out[e] = sum of entry e's partial sums, in pairs of pairs of chunks: a wave an entry.
__global__ __launch_bounds__(256) void k_project_sum(int ne, int npart, int g, const double* __restrict__ partial,
                                                     double* __restrict__ out) {
    constexpr int GROUPS = PJ_CHUNKS / PJ_GROUP;
    const int lane = threadIdx.x & 63;
    const long long e = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (e >= ne) return;  // uniform in the wave
    const double* p = partial + e * npart;
    auto at = [&](int i) { return i < npart ? p[i] : 0.0; };
    double s = 0.0;
#pragma unroll
    for (int h = 0; h < GROUPS / 64; ++h) {
        const int c = lane + 64 * h;
        s += g == 4 ? at(c) : g == 2 ? at(2 * c) + at(2 * c + 1)
                                     : (at(4 * c) + at(4 * c + 1)) + (at(4 * c + 2) + at(4 * c + 3));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) out[e] = s;
}

// W[a][q] = sum_s psi[s][q] v[a * nocc + s][q]
__global__ __launch_bounds__(256) void k_cross_w(long long ndof, int nu, int nocc, const double* __restrict__ psi,
                                                 const double* __restrict__ v, double* __restrict__ W) {
    const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
    const int a = blockIdx.y;
    if (q >= ndof || a >= nu) return;
    double s = 0.0;
    for (int k = 0; k < nocc; ++k) s += psi[(long long)k * ndof + q] * v[((long long)a * nocc + k) * ndof + q];
    W[(long long)a * ndof + q] = s;
}

// rho[a * nocc + s] = u[a] psi[s] on every node
__global__ __launch_bounds__(256) void k_cross_products(long long ndof, int nu, int nocc,
                                                        const double* __restrict__ u, const double* __restrict__ psi,
                                                        double* __restrict__ rho) {
    const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
    const int pr = blockIdx.y, a = pr / nocc, s = pr % nocc;
    if (q >= ndof || a >= nu) return;
    rho[(long long)pr * ndof + q] = u[(long long)a * ndof + q] * psi[(long long)s * ndof + q];
}

// One work-group: M (nocc x nocc, row-major, M[k][l] = (psi_k, W_l)) -> its symmetric part,
// the Cholesky factor L (M = L L^T) and T = L^-1 (lower triangular, written row-major).
// flag[0] = 1 when a pivot is not positive (M not positive definite); T is then not to be used.
constexpr int ACE_MAX = 64;
__global__ __launch_bounds__(256) void k_ace_factor(int n, const double* __restrict__ Min, double* __restrict__ T,
                                                    int* flag) {
    __shared__ double L[ACE_MAX][ACE_MAX + 1];
    __shared__ double Ti[ACE_MAX][ACE_MAX + 1];
    __shared__ int bad;
    const int t = threadIdx.x;
    if (t == 0) bad = 0;
    for (int e = t; e < n * n; e += 256) {
        const int r = e / n, c = e % n;
        L[r][c] = 0.5 * (Min[r * n + c] + Min[c * n + r]);
    }
    __syncthreads();
    for (int j = 0; j < n; ++j) {  // column j: pivot, then the entries below it
        if (t == 0) {
            double d = L[j][j];
            for (int k = 0; k < j; ++k) d -= L[j][k] * L[j][k];
            if (!(d > 0.0)) {
                bad = 1;
                d = 1.0;
            }
            L[j][j] = sqrt(d);
        }
        __syncthreads();
        for (int r = j + 1 + t; r < n; r += 256) {
            double s = L[r][j];
            for (int k = 0; k < j; ++k) s -= L[r][k] * L[j][k];
            L[r][j] = s / L[j][j];
        }
        __syncthreads();
    }
    // T = L^-1, one column per thread by forward substitution on e_c
    for (int c = t; c < n; c += 256) {
        for (int r = 0; r < n; ++r) {
            if (r < c) {
                Ti[r][c] = 0.0;
                continue;
            }
            double s = (r == c) ? 1.0 : 0.0;
            for (int k = c; k < r; ++k) s -= L[r][k] * Ti[k][c];
            Ti[r][c] = s / L[r][r];
        }
    }
    __syncthreads();
    for (int e = t; e < n * n; e += 256) T[e] = Ti[e / n][e % n];
    if (t == 0) flag[0] = bad;
}

// xi[k][q] = sum_{j <= k} T[k][j] W[j][q]
__global__ __launch_bounds__(256) void k_ace_combine(long long ndof, int n, const double* __restrict__ T,
                                                     const double* __restrict__ W, double* __restrict__ xi) {
    __shared__ double Ts[ACE_MAX * ACE_MAX];
    for (int e = threadIdx.x; e < n * n; e += 256) Ts[e] = T[e];
    __syncthreads();
    const long long q = (long long)blockIdx.x * 256 + threadIdx.x;
    if (q >= ndof) return;
    for (int k = 0; k < n; ++k) {  // W[j][q] is re-read per k from L1/L2: this step runs once per SCF rebuild
        double s = 0.0;
        for (int j = 0; j <= k; ++j) s += Ts[k * n + j] * W[(long long)j * ndof + q];
        xi[(long long)k * ndof + q] = s;
    }
}

// C[i][a] = sum_k A[i][k] B[k][a]  (small dense product, one thread per output)
__global__ __launch_bounds__(256) void k_small_gemm(int ni, int nk, int na, const double* __restrict__ A,
                                                    const double* __restrict__ B, double* __restrict__ C) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= ni * na) return;
    const int i = e / na, a = e % na;
    double s = 0.0;
    for (int k = 0; k < nk; ++k) s += A[(long long)i * nk + k] * B[(long long)k * na + a];
    C[e] = s;
}

}  // namespace

// Rows of phi of a work-group: 64, or 16 for a few rows (the compressed exchange's overlaps, 8 x 8),
// where a launch needs the work-groups more than the saved reads of u.
static int project_rows(int nbasis) { return nbasis > 16 ? 64 : 16; }

// Nodes of a chunk, in whole steps of the work-group's four waves.
static long long project_nodes(long long ndof) {
    return std::max(256LL, ((ndof + PJ_CHUNKS - 1) / PJ_CHUNKS + 63) / 64 * 64);
}
static long long project_chunks(long long ndof) { return (ndof + project_nodes(ndof) - 1) / project_nodes(ndof); }

// Chunks of a work-group: as many as leave the launch about 512 work-groups.
static int project_group(int nbasis, int nu) {
    const int rows = project_rows(nbasis);
    const long long tiles = (long long)((nbasis + rows - 1) / rows) * ((nu + 15) / 16);
    return tiles >= 4 ? 4 : tiles >= 2 ? 2 : 1;
}
static int project_parts(long long ndof, int g) { return (int)((project_chunks(ndof) + g - 1) / g); }

// Rows of phi of a launch: all, or whole tiles whose partial sums fit.
static int project_pass(long long ndof, int nbasis, int nu) {
    const long long rows = PJ_PARTIAL / ((long long)nu * project_parts(ndof, project_group(nbasis, nu))) / 64 * 64;
    return (int)std::min<long long>(nbasis, std::max(64LL, rows));
}

long long project_partials(long long ndof, int nbasis, int nu) {
    return (long long)project_pass(ndof, nbasis, nu) * project_parts(ndof, project_group(nbasis, nu)) * nu;
}

void launch_project(const LevelHost& L, int nbasis, const double* phi, int nu, const double* u, const double* f,
                    double* partial, double* out, hipStream_t s) {
    if (nbasis == 0 || nu == 0) return;
    if (L.ndof >= 0x7fffffffLL || L.n * L.n * L.n > PJ_MAXN3) throw std::runtime_error("projection: field too large");
    const int g = project_group(nbasis, nu), npart = project_parts(L.ndof, g), cn = (int)project_nodes(L.ndof);
    const int pass = project_pass(L.ndof, nbasis, nu);
    for (int i = 0; i < nbasis; i += pass) {
        const int nb = std::min(pass, nbasis - i), rows = project_rows(nb);
        const long long grid = (long long)((nb + rows - 1) / rows) * ((nu + 15) / 16) * npart;
        if (grid > 0x7fffffffLL) throw std::runtime_error("projection grid too large");
        auto* k = rows == 64 ? k_project<4> : k_project<1>;
        hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(PJ_THREADS), 0, s, L.dev64, L.n, (int)L.ndof, nb,
                           phi + i * L.ndof, nu, u, f, npart, g, cn, partial);
        hipLaunchKernelGGL(k_project_sum, dim3((unsigned)((nb * nu + 3) / 4)), dim3(256), 0, s, nb * nu, npart, g, partial,
                           out + (long long)i * nu);
    }
}

void launch_cross_products(long long ndof, int nu, int nocc, const double* u, const double* psi, double* rho,
                           hipStream_t s) {
    if (nu == 0 || nocc == 0) return;
    hipLaunchKernelGGL(k_cross_products, dim3((unsigned)((ndof + 255) / 256), nu * nocc), dim3(256), 0, s, ndof, nu,
                       nocc, u, psi, rho);
}

void launch_cross_w(long long ndof, int nu, int nocc, const double* psi, const double* v, double* W, hipStream_t s) {
    if (nu == 0) return;
    hipLaunchKernelGGL(k_cross_w, dim3((unsigned)((ndof + 255) / 256), nu), dim3(256), 0, s, ndof, nu, nocc, psi, v, W);
}

void launch_ace_factor(int n, const double* M, double* T, int* flag, hipStream_t s) {
    if (n < 1 || n > ACE_MAX) throw std::runtime_error("ACE: bad orbital count");
    hipLaunchKernelGGL(k_ace_factor, dim3(1), dim3(256), 0, s, n, M, T, flag);
}

void launch_ace_combine(long long ndof, int n, const double* T, const double* W, double* xi, hipStream_t s) {
    hipLaunchKernelGGL(k_ace_combine, dim3((unsigned)((ndof + 255) / 256)), dim3(256), 0, s, ndof, n, T, W, xi);
}

void launch_small_gemm(int ni, int nk, int na, const double* A, const double* B, double* C, hipStream_t s) {
    if (ni * na == 0) return;
    hipLaunchKernelGGL(k_small_gemm, dim3((unsigned)((ni * na + 255) / 256)), dim3(256), 0, s, ni, nk, na, A, B, C);
}

}  // namespace dg
