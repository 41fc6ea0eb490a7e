// Dirichlet data of the auxiliary-mesh Poisson problem by quadrature (Sec. 6.3).
//
// The full-space problem -Lap u = 4 pi f is restated on the mesh domain with
// Dirichlet data equal to the Coulomb potential of f on the boundary, and that
// integral is evaluated with the quadrature rule of the mesh's own nodal grid
// (here the GLL grid, whose weights are the lumped mass W_q):
//
//     g(r) = sum_q W_q f(x_q) / |r - x_q|      for every boundary node r.
//
// Every boundary node is itself a grid node (and, on an element face, also the
// node of the neighbouring element at the same place), where the integrand is
// singular; the method has f vanish there, so terms closer than a millionth of
// the smallest element width are left out.
//
// Reflections.  The mesh is uniform, so its nodes, weights and boundary nodes are
// invariant under the eight reflections rho of the box about its centre, and the
// sum is a convolution over that group: with b and a running over one octant of the
// boundary and of the grid, chi_s the eight parities, and
//     F_s(a) = sum_sigma chi_s(sigma) (W f)(sigma a),
//     K_s(b, a) = sum_tau chi_s(tau) / |b - tau a|,
// g(rho b) = 1/8 sum_s chi_s(rho) sum_a K_s(b, a) F_s(a).  A pair (b, a) costs eight
// inverse distances and 8 multiply-adds per source where the plain sum over its 64
// images costs 64 of each: an eighth of the work, with the same terms in FP64.  (Rounding is that of the
// largest of the eight images' values: for densities over the grid that of the plain sum, 2e-13; for a single node's
// value by one end of 32 x 4 x 4 elements 1.5e-15 of the largest datum against 1.3e-16, and at the far end 1e-14
// of the datum itself against 3e-16.)
// (A node whose coordinate is its own mirror image, the middle one of an odd count,
// is met twice by the group; its weight is halved per such axis.)
//
// The sum is bound by FP64 issue (vector and matrix units share the 72-78 TFLOP/s):
//  * k_quad_pack writes, for a tile of R sources, the records F_s(a) as [a][s][R] in
//    lattice order of the octant;
//  * k_quad (R <= 4): a lane owns one octant boundary node and its 8 R sums; all lanes
//    visit the grid nodes in the same order, so the records are wave-uniform and come
//    in through scalar loads as SGPR operands of the FMAs;
//  * k_quad_mfma (R = 16, 32): per parity a matrix product K_s F_s on
//    v_mfma_f64_16x16x4; a lane computes the eight inverse distances of one
//    (boundary node, grid node) pair and their parity combinations, which are its A
//    operands as they are, and the records are staged in LDS for the work-group's
//    four waves (64 boundary nodes);
//  * k_quad_combine adds the split parts in a fixed order and turns the eight parity
//    sums of an octant boundary node into the values at its eight images.
// The octant is split into parts so that a launch holds several rounds of resident
// waves; work-groups are ordered so that each XCD takes the boundary tiles of one part
// at a time: they stream the same records through its L2.
//
// Measured (36 pair densities of 16^3 elements, p = 4; 38,400 boundary nodes x 512,000
// grid nodes): 6.0 ms for the whole call, 33.5 ms as a plain sum over all nodes; one density
// 1.26 ms against 6.8.  16 sources take 2.7 ms, 4 1.6: a pass costs about 1.2 ms of
// inverse distances (83 FP64 instructions and 8 reciprocal roots per pair) and 0.10 ms a source (of
// the padded width on the matrix unit); the FP64 vector and matrix instructions do not
// overlap, so the sum of the two bounds it.
// Tried: 48 and 64 sources a tile (one wave per SIMD: 9.7 and 28 ms), K of the next step formed
// between the matrix instructions (no faster).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <stdexcept>
#include <type_traits>

#include "dg_internal.h"
#include "dg_kernels.h"

namespace dg {

namespace {

constexpr int QUAD_BLOCK = 256;    // threads per work-group
constexpr int QUAD_VEC = 4;        // widest source tile of the vector kernel
// Source tile for `left` more sources, at most rmax.  Up to 4 go to the vector kernel (1.3 to 1.6 ms on 16^3
// elements, p = 4, against 2.6 ms for a matrix tile of 16; its records then fill the SGPRs), more to the
// narrowest matrix tile that holds them (17 to 20 sources: 4.30 ms in a tile of 32; 16 and a vector pass of 1, 2
// or 4 would take 4.06, 4.18 and 4.32).
constexpr int quad_tile(int left, int rmax) {
    if (left > 16 && rmax >= 32) return 32;
    if (left > QUAD_VEC && rmax >= 16) return 16;
    return left < QUAD_VEC ? (left < rmax ? left : rmax) : (rmax < QUAD_VEC ? rmax : QUAD_VEC);
}
// Parts the octant is split into: 64, of at least 80 nodes, and fewer where the boundary alone gives the waves
// (of 64 octant boundary nodes).  One number for both kernels (quad_parts).  The whole call with 48 / 64 / 80 / 100
// parts, and before with 8,192 work-group waves for the matrix kernel and 16,384 for the vector kernel: 16^3
// elements p = 4, 1 source 1.30 / 1.26 / 1.25 / 1.35 ms (1.50), 16 sources 2.75 / 2.69 / 2.78 / 2.89 (2.77), 36
// 6.11 / 5.98 / 6.08 / 6.31 (6.48); 8^3 x 8 0.23 / 0.26 / 0.29 / 0.35 (0.35); 12^3 x 1 0.50 / 0.45 / 0.49 / 0.53
// (0.98); 20^3 x 2 3.93 / 3.91 / 3.91 / 3.90 (3.81); 24^3 x 3 10.7 / 9.8 / 10.1 / 10.1 (9.9); 32^3 x 12, cut by
// the waves, 73 (87; at 4,096 waves 81).
constexpr int QUAD_PARTS = 64, QUAD_PART_NODES = 80, QUAD_WAVES = 12288;
constexpr int QUAD_CHUNK = 8;      // octant nodes per LDS stage of the matrix kernel (two MFMA steps)

typedef double v4d __attribute__((ext_vector_type(4)));

// Octant sizes: node counts per axis N and of the half axes H = ceil(N / 2).
struct QuadDims {
    int N[3], H[3];
    int noct;   // octant grid nodes
    int nbo;    // octant boundary nodes (faces x, y, z in turn)
};

QuadDims quad_dims(const LevelHost& L) {
    QuadDims d;
    for (int k = 0; k < 3; ++k) {
        d.N[k] = L.E[k] * L.n;
        d.H[k] = (d.N[k] + 1) / 2;
    }
    d.noct = d.H[0] * d.H[1] * d.H[2];
    d.nbo = d.H[2] * d.H[1] + d.H[2] * d.H[0] + d.H[1] * d.H[0];
    return d;
}

// sum over parities: v[s] = sum_t chi_s(t) v[t], bit d of the index standing for axis d
__device__ __forceinline__ void parities(double (&v)[8]) {
#pragma unroll
    for (int d = 1; d < 8; d <<= 1)
#pragma unroll
        for (int t = 0; t < 8; ++t)
            if (!(t & d)) {
                const double a = v[t], b = v[t | d];
                v[t] = a + b;
                v[t | d] = a - b;
            }
}

// octant boundary node -> lattice indices (all in the lower half)
__device__ __forceinline__ void oct_face_node(int b, const QuadDims& D, int& f, int& X, int& Y, int& Z) {
    const int fx = D.H[2] * D.H[1], fy = D.H[2] * D.H[0];
    if (b < fx) {
        f = 0; X = 0; Y = b % D.H[1]; Z = b / D.H[1];
    } else if (b < fx + fy) {
        b -= fx;
        f = 1; Y = 0; X = b % D.H[0]; Z = b / D.H[0];
    } else {
        b -= fx + fy;
        f = 2; Z = 0; X = b % D.H[0]; Y = b / D.H[0];
    }
}

// where the image rho of that node lies in a face vector (x faces [Z][Y], y faces [Z][X], z faces [Y][X])
__device__ __forceinline__ int face_slot(int f, int X, int Y, int Z, int rho, const QuadDims& D) {
    const int NX = D.N[0], NY = D.N[1], NZ = D.N[2];
    const int x = rho & 1 ? NX - 1 - X : X, y = rho & 2 ? NY - 1 - Y : Y, z = rho & 4 ? NZ - 1 - Z : Z;
    if (f == 0) return (rho & 1) * NZ * NY + z * NY + y;
    if (f == 1) return 2 * NZ * NY + ((rho >> 1) & 1) * NZ * NX + z * NX + x;
    return 2 * NZ * NY + 2 * NZ * NX + ((rho >> 2) & 1) * NY * NX + y * NX + x;
}

// axes (bits) on which the node is its own mirror image
__device__ __forceinline__ int self_mask(int X, int Y, int Z, const QuadDims& D) {
    return (2 * X == D.N[0] - 1 ? 1 : 0) | (2 * Y == D.N[1] - 1 ? 2 : 0) | (2 * Z == D.N[2] - 1 ? 4 : 0);
}

// one source value W f at a lattice node
__device__ __forceinline__ double quad_source(int s, int X, int Y, int Z, const QuadDims& D, int n, long long ndof,
                                              const LevelDev<double>* __restrict__ dev,
                                              const double* __restrict__ f, const double* __restrict__ phi,
                                              const int* __restrict__ pi, const int* __restrict__ pj) {
    const int ex = X / n, i = X - ex * n, ey = Y / n, j = Y - ey * n, ez = Z / n, k = Z - ez * n;
    const long long q = (((long long)ez * (D.N[1] / n) + ey) * (D.N[0] / n) + ex) * (n * n * n) + (k * n + j) * n + i;
    const double w = dev->ax[0].m[i] * dev->ax[1].m[j] * dev->ax[2].m[k];
    return w * (f ? f[(long long)s * ndof + q] : phi[(long long)pi[s] * ndof + q] * phi[(long long)pj[s] * ndof + q]);
}

// Records F_s(a), [a][s][R].  A work-group takes 16 octant nodes (runs of neighbouring nodes) and 16
// sources at a time; the records leave through LDS so that both sides are contiguous.
constexpr int PACK_NODES = 16, PACK_SRC = 16;
__global__ __launch_bounds__(PACK_NODES* PACK_SRC) void k_quad_pack(const LevelDev<double>* __restrict__ dev,
                                                                    QuadDims D, int n, long long ndof, int nsrc,
                                                                    int r0, int R, const double* __restrict__ f,
                                                                    const double* __restrict__ phi,
                                                                    const int* __restrict__ pi,
                                                                    const int* __restrict__ pj,
                                                                    double* __restrict__ rec) {
    __shared__ double out[PACK_NODES][8][PACK_SRC];
    const int q0 = blockIdx.x * PACK_NODES, nn = min(PACK_NODES, D.noct - q0);
    const int a = threadIdx.x % PACK_NODES, r = threadIdx.x / PACK_NODES;
    const int q = min(q0 + a, D.noct - 1);
    const int X = q % D.H[0], Y = (q / D.H[0]) % D.H[1], Z = q / (D.H[0] * D.H[1]);
    const int self = self_mask(X, Y, Z, D);
    const double half = 1.0 / (double)(1 << __popc(self));
    for (int rb = 0; rb < R; rb += PACK_SRC) {
        const int s = r0 + rb + r, nr = min(PACK_SRC, R - rb);
        double v[8];
#pragma unroll
        for (int t = 0; t < 8; ++t)
            v[t] = s < nsrc && rb + r < R
                       ? half * quad_source(s, t & 1 ? D.N[0] - 1 - X : X, t & 2 ? D.N[1] - 1 - Y : Y,
                                            t & 4 ? D.N[2] - 1 - Z : Z, D, n, ndof, dev, f, phi, pi, pj)
                       : 0.0;
        parities(v);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 8; ++t) out[a][t][r] = v[t];
        __syncthreads();
        for (int t = threadIdx.x; t < nn * 8 * nr; t += PACK_NODES * PACK_SRC) {
            const int row = t / nr, c = t - row * nr;
            rec[((long long)q0 * 8 + row) * R + rb + c] = out[row / 8][row % 8][c];
        }
    }
}

// 1/sqrt(r2); with MASK, 0 for a node at the boundary node itself.
template <bool MASK>
__device__ __forceinline__ double inv_dist(double r2, double drop2) {
    // the hardware estimate is good to about 5e-8; with e = 1 - r2 y^2 the exact value is
    // y (1 - e)^(-1/2) = y (1 + e/2 + 3e^2/8 + ...), so two terms of the series leave O(e^3)
    double y = __builtin_amdgcn_rsq(r2);
    const double e = fma(-(r2 * y), y, 1.0);
    y = fma(y * e, fma(0.375, e, 0.5), y);
    if (MASK) y = r2 > drop2 ? y : 0.0;
    return y;
}

// K_s of a pair: d[t] = squared distance in y and z to the images (ty, tz) = (t & 1, t >> 1), and the
// distances of the two x images from the boundary node's and the grid node's distance to the centre.
template <bool MASK>
__device__ __forceinline__ void pair_kernel(double bx, double ax, const double (&d)[4], double drop2,
                                            double (&k)[8]) {
    const double xm = bx - ax, xp = bx + ax;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        k[2 * t] = inv_dist<MASK>(fma(xm, xm, d[t]), drop2);
        k[2 * t + 1] = inv_dist<MASK>(fma(xp, xp, d[t]), drop2);
    }
    parities(k);
}

__device__ __forceinline__ void yz_dist(double by, double bz, double ay, double az, double (&d)[4]) {
    const double ym = by - ay, yp = by + ay, zm = bz - az, zp = bz + az;
    const double zm2 = zm * zm, zp2 = zp * zp;
    d[0] = fma(ym, ym, zm2);
    d[1] = fma(yp, yp, zm2);
    d[2] = fma(ym, ym, zp2);
    d[3] = fma(yp, yp, zp2);
}

// Work-groups are dispatched to the eight XCDs round robin (w % 8).  Give XCD x a contiguous
// range of the logical work-group order, in which consecutive work-groups are the boundary
// tiles of one part of the octant: the tiles in flight on an XCD then stream the same
// records through its L2.
__device__ __forceinline__ int quad_xcd_remap(int w, int G) {
    constexpr int NXCD = 8;
    if (G < NXCD) return w;
    const int x = w % NXCD, slot = w / NXCD;
    const int base = G / NXCD, rem = G % NXCD;
    return x * base + min(x, rem) + slot;
}

// distances from the centre of the box of lattice node X and its axis table
__device__ __forceinline__ double centred(const double* __restrict__ x, int N, int X) {
    return 0.5 * (x[0] + x[N - 1]) - x[X];
}

// Parity sums of the octant boundary node: slot of image s in the part's face vector.  A parity that is
// odd on an axis where the node is its own image has a zero sum and no slot of its own.
__device__ __forceinline__ void store_parity(double* __restrict__ o, int b, int s, const QuadDims& D, double v) {
    int f, X, Y, Z;
    oct_face_node(b, D, f, X, Y, Z);
    if (!(s & self_mask(X, Y, Z, D))) o[face_slot(f, X, Y, Z, s, D)] = v;
}

template <int R>
__global__ __launch_bounds__(QUAD_BLOCK) void k_quad(const double* __restrict__ xs, const double* __restrict__ ys,
                                                     const double* __restrict__ zs, QuadDims D, int nface, int nper,
                                                     int ntb, double drop2, const double* __restrict__ rec,
                                                     double* __restrict__ out) {
    // logical work-group: boundary tile (fastest) and part of the octant
    const int w = quad_xcd_remap(blockIdx.x, gridDim.x);
    const int tile = w % ntb, part = w / ntb;
    const int b = tile * QUAD_BLOCK + threadIdx.x;
    int f, X, Y, Z;
    oct_face_node(min(b, D.nbo - 1), D, f, X, Y, Z);
    const double bx = centred(xs, D.N[0], X), by = centred(ys, D.N[1], Y), bz = centred(zs, D.N[2], Z);
    double acc[8][R];
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[s][r] = 0.0;
    const double cx = 0.5 * (xs[0] + xs[D.N[0] - 1]);
    int q = part * nper;
    const int q1 = min(D.noct, q + nper);
    auto pair = [&](auto mask, const double (&d)[4], double ax, const double* __restrict__ F) {
        double k[8];
        pair_kernel<decltype(mask)::value>(bx, ax, d, drop2, k);
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int r = 0; r < R; ++r) acc[s][r] = fma(F[s * R + r], k[s], acc[s][r]);
    };
    while (q < q1) {
        // the rest of one lattice row; only rows on the boundary surface, and the first node of any
        // other row, can meet the boundary node itself
        const int row = q / D.H[0], x0 = q - row * D.H[0], x1 = min(D.H[0], x0 + q1 - q);
        const int yq = row % D.H[1], zq = row / D.H[1];
        double d[4];
        yz_dist(by, bz, centred(ys, D.N[1], yq), centred(zs, D.N[2], zq), d);
        const double* F = rec + (long long)row * D.H[0] * (8 * R);
        const int m1 = yq == 0 || zq == 0 ? x1 : min(x1, max(x0, 1));
        int x = x0;
        for (; x < m1; ++x) pair(std::true_type{}, d, cx - xs[x], F + (long long)x * (8 * R));
#pragma unroll 2
        for (; x < x1; ++x) pair(std::false_type{}, d, cx - xs[x], F + (long long)x * (8 * R));
        q += x1 - x0;
    }
    if (b >= D.nbo) return;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int s = 0; s < 8; ++s) store_parity(out + ((long long)part * R + r) * nface, b, s, D, acc[s][r]);
}

// R = 16 NT sources: a wave owns 16 octant boundary nodes, a work-group 64.
template <int NT>
__global__ __launch_bounds__(QUAD_BLOCK, 2) void k_quad_mfma(const double* __restrict__ xs,
                                                             const double* __restrict__ ys,
                                                             const double* __restrict__ zs, QuadDims D, int nface,
                                                             int nper, int ntb, double drop2,
                                                             const double* __restrict__ rec,
                                                             double* __restrict__ out, int nr) {
    constexpr int R = 16 * NT, NV = 8 * R;               // values of a node's record
    constexpr int NS = NV + 16;                          // its LDS stride: two nodes fall on different banks
    constexpr int LD = QUAD_CHUNK * NV / (2 * QUAD_BLOCK);  // double2 a thread stages per chunk
    static_assert(LD * 2 * QUAD_BLOCK == QUAD_CHUNK * NV, "chunk is not a whole number of loads");
    __shared__ double sF[2][QUAD_CHUNK * NS];
    const int w = quad_xcd_remap(blockIdx.x, gridDim.x);
    const int tile = w % ntb, part = w / ntb;
    const int t = threadIdx.x, lane = t & 63, m = lane & 15, kq = lane >> 4;
    const int b0 = tile * 64 + (t >> 6) * 16;
    int f, X, Y, Z;
    oct_face_node(min(b0 + m, D.nbo - 1), D, f, X, Y, Z);
    const double bx = centred(xs, D.N[0], X), by = centred(ys, D.N[1], Y), bz = centred(zs, D.N[2], Z);
    const double cx = 0.5 * (xs[0] + xs[D.N[0] - 1]), cy = 0.5 * (ys[0] + ys[D.N[1] - 1]),
                 cz = 0.5 * (zs[0] + zs[D.N[2] - 1]);
    v4d acc[8][NT];
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[s][n] = v4d{0.0, 0.0, 0.0, 0.0};
    const int q0 = part * nper, q1 = min(D.noct, q0 + nper);
    const long long vend = (long long)q1 * NV;  // records end here; a last chunk is filled up with zeros
    double2 st[LD];
    auto stage_load = [&](int q) {
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const long long v = (long long)q * NV + 2 * (i * QUAD_BLOCK + t);
            st[i] = v < vend ? *reinterpret_cast<const double2*>(rec + v) : double2{0.0, 0.0};
        }
    };
    auto stage_store = [&](int buf) {
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const int v = 2 * (i * QUAD_BLOCK + t);
            *reinterpret_cast<double2*>(&sF[buf][(v / NV) * NS + v % NV]) = st[i];
        }
    };
    // the lane's grid node (x fastest), advanced by four nodes per MFMA step; past the end it stays on the
    // last plane, where its record is zero
    const int HX = D.H[0], HY = D.H[1], HZ = D.H[2];
    int xq, yq, zq;
    {
        const int q = q0 + kq;
        xq = q % HX;
        yq = (q / HX) % HY;
        zq = q / (HX * HY);
    }
    stage_load(q0);
    stage_store(0);
    int buf = 0;
    for (int q = q0; q < q1; q += QUAD_CHUNK, buf ^= 1) {
        __syncthreads();  // this chunk is staged; the other buffer's readers are done
        const bool more = q + QUAD_CHUNK < q1;
        if (more) stage_load(q + QUAD_CHUNK);
#pragma unroll
        for (int step = 0; step < QUAD_CHUNK / 4; ++step) {
            double d[4], k[8];
            const int zc = min(zq, HZ - 1);
            yz_dist(by, bz, cy - ys[yq], cz - zs[zc], d);
            const double ax = cx - xs[xq];
            if (__any(xq == 0 || yq == 0 || zc == 0))
                pair_kernel<true>(bx, ax, d, drop2, k);
            else
                pair_kernel<false>(bx, ax, d, drop2, k);
            const double* F = &sF[buf][(step * 4 + kq) * NS + m];
#pragma unroll
            for (int s = 0; s < 8; ++s)
#pragma unroll
                for (int n = 0; n < NT; ++n)
                    acc[s][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(k[s], F[s * R + n * 16], acc[s][n], 0, 0, 0);
            xq += 4;
            while (xq >= HX) {
                xq -= HX;
                if (++yq == HY) {
                    yq = 0;
                    ++zq;
                }
            }
        }
        if (more) stage_store(buf ^ 1);
    }
    // accumulator: source = lane & 15, boundary node = lane / 16 + 4 * register
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int b = b0 + kq + 4 * i;
        if (b >= D.nbo) continue;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            if (n * 16 + m >= nr) continue;
#pragma unroll
            for (int s = 0; s < 8; ++s)
                store_parity(out + ((long long)part * nr + n * 16 + m) * nface, b, s, D, acc[s][n][i]);
        }
    }
}

// g at the eight images of an octant boundary node from its parity sums (S parts, face vectors `stride`
// sources apart; part and g may be the same vectors).  Grid (octant boundary nodes / 256, sources).
//
// A source with a value that is not finite has parity sums that are not finite either; its data are then
// what the plain sum over all nodes gives (an infinite value stays one, rather than infinity minus infinity
// between mirror images).  Every inverse distance is positive but the dropped one of the boundary node itself,
// so that sum is infinite where the infinite terms have one sign, and NaN where they have two, where a term is
// NaN or where the node's own term is infinite (0 times infinity).  The work-group looks through the source's
// values together: 0.5 to 1.4 ms more for 512,000 nodes (a lane that walked the grid by itself would take a
// dependent step a node).
__global__ __launch_bounds__(256) void k_quad_combine(const double* part, int S, int R, QuadDims D, int nface, int r0,
                                                      const LevelDev<double>* __restrict__ dev, int n, long long ndof,
                                                      const double* __restrict__ xs, const double* __restrict__ ys,
                                                      const double* __restrict__ zs, double drop2,
                                                      const double* __restrict__ f, const double* __restrict__ phi,
                                                      const int* __restrict__ pi, const int* __restrict__ pj,
                                                      double* g) {
    constexpr int POS = 1, NEG = 2, NAN_ = 4;
    __shared__ int terms;
    const int r = blockIdx.y, src = r0 + r, own = blockIdx.x * 256 + threadIdx.x, b = min(own, D.nbo - 1);
    int fc, X, Y, Z;
    oct_face_node(b, D, fc, X, Y, Z);
    const int self = self_mask(X, Y, Z, D);
    double v[8];
    bool finite = true;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int slot = face_slot(fc, X, Y, Z, s, D);
        double a = 0.0;
        if (!(s & self))
            for (int p = 0; p < S; ++p) a += part[((long long)p * R + r) * nface + slot];
        v[s] = a;
        finite &= isfinite(a);
    }
    parities(v);
    if (threadIdx.x == 0) terms = 0;
    if (__syncthreads_or(!finite)) {
        const double *fa = f ? f + src * ndof : phi + pi[src] * ndof, *fb = f ? nullptr : phi + pj[src] * ndof;
        int mine = 0;
#pragma unroll 4
        for (long long q = threadIdx.x; q < ndof; q += 256) {
            double a = fa[q];
            if (fb) a *= fb[q];
            if (fabs(a) < 1e200) continue;  // the product with its weight is finite
            const int n3 = n * n * n, l = (int)(q % n3);
            a *= dev->ax[0].m[l % n] * dev->ax[1].m[l / n % n] * dev->ax[2].m[l / (n * n)];
            mine |= isnan(a) ? NAN_ : !isinf(a) ? 0 : a > 0.0 ? POS : NEG;
        }
        if (mine) atomicOr(&terms, mine);
        __syncthreads();
        if (terms && !finite) {
            const double inf = terms == POS ? INFINITY : terms == NEG ? -INFINITY : NAN;
            for (int s = 0; s < 8; ++s) {
                const int x0 = s & 1 ? D.N[0] - 1 - X : X, y0 = s & 2 ? D.N[1] - 1 - Y : Y,
                          z0 = s & 4 ? D.N[2] - 1 - Z : Z;
                v[s] = inf;
                // the nodes at the same place: the node itself and those of the neighbour elements
                for (int z = max(z0 - 1, 0); z <= min(z0 + 1, D.N[2] - 1); ++z)
                    for (int y = max(y0 - 1, 0); y <= min(y0 + 1, D.N[1] - 1); ++y)
                        for (int x = max(x0 - 1, 0); x <= min(x0 + 1, D.N[0] - 1); ++x) {
                            const double dx = xs[x0] - xs[x], dy = ys[y0] - ys[y], dz = zs[z0] - zs[z];
                            if (!(fma(dx, dx, fma(dy, dy, dz * dz)) > drop2) &&
                                isinf(quad_source(src, x, y, z, D, n, ndof, dev, f, phi, pi, pj)))
                                v[s] = NAN;
                        }
            }
        }
    }
    if (own >= D.nbo) return;
#pragma unroll
    for (int s = 0; s < 8; ++s) g[(long long)src * nface + face_slot(fc, X, Y, Z, s, D)] = 0.125 * v[s];
}

}  // namespace

// Work space of the entry point that allocates nothing (dg_boundary_data_noalloc): the packed
// records and the split partial sums live in this array, one copy per GPU, kept until the
// process ends.  Host code never uses its name as an address: quad_scratch_init looks up each
// device's copy once and quad_scratch returns it.  Every call on a GPU shares that GPU's copy.
constexpr long long QUAD_SCRATCH_DOUBLES = 8LL << 20;  // 64 MiB
static __device__ __align__(256) double scratch[QUAD_SCRATCH_DOUBLES];

namespace {
constexpr int QUAD_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
double* g_scratch[QUAD_MAX_DEVICES] = {};
}  // namespace

hipError_t quad_scratch_init(int device) {
    if (device < 0 || device >= QUAD_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch[device]) return hipSuccess;
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch[device] = static_cast<double*>(p);
    return hipSuccess;
}

double* quad_scratch(int device, long long* capacity) {
    if (capacity) *capacity = QUAD_SCRATCH_DOUBLES;
    if (device < 0 || device >= QUAD_MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    return g_scratch[device];
}

namespace {

// Parts of the octant: by the mesh alone, so that a source's data do not depend on the others of its call.
// (v_mfma_f64_16x16x4 adds its four products one after the other, each rounded as a fused multiply-add: the
// vector and the matrix kernel give the same sums of a part, bit for bit.)
int quad_parts(const QuadDims& D) {
    const int waves = (D.nbo + 63) / 64;
    return std::max(1, std::min({D.noct / QUAD_PART_NODES, QUAD_PARTS, QUAD_WAVES / waves}));
}

// One pass over the octant: source tile, the sources in it, nodes per part, parts (at most `most`).  One part
// leaves its sums in g itself.
struct QuadPass {
    int R, nr, nper, S;
};
QuadPass quad_pass(const QuadDims& D, int left, int rmax, long long part_len, long long nface) {
    QuadPass T{};
    T.R = quad_tile(left, rmax);
    T.nr = std::min(T.R, left);
    const long long most = std::max(1LL, std::min<long long>(quad_parts(D), part_len / (T.nr * nface)));
    const int nper = (int)((D.noct + most - 1) / most);
    T.nper = (nper + QUAD_CHUNK - 1) / QUAD_CHUNK * QUAD_CHUNK;
    T.S = (D.noct + T.nper - 1) / T.nper;
    return T;
}

// The plan with source tiles of at most rmax in `capacity` doubles; rmax = 0 when it does not fit.
QuadPlan quad_plan_width(const LevelHost& L, int nsrc, int rmax, long long capacity) {
    const QuadDims D = quad_dims(L);
    QuadPlan P{};
    P.nface = 2 * ((long long)D.N[2] * D.N[1] + (long long)D.N[2] * D.N[0] + (long long)D.N[1] * D.N[0]);
    for (int left = nsrc; left > 0; left -= quad_tile(left, rmax)) {
        const int R = quad_tile(left, rmax);
        P.rec_len = std::max(P.rec_len, 8LL * D.noct * R);
        P.part_len = std::max(P.part_len, (long long)quad_parts(D) * std::min(R, left) * P.nface);
    }
    if (P.rec_len > capacity) return P;
    P.part_len = std::min(P.part_len, capacity - P.rec_len);
    P.wgs = 1LL << 40;
    for (int left = nsrc; left > 0; left -= quad_tile(left, rmax)) {
        const QuadPass T = quad_pass(D, left, rmax, P.part_len, P.nface);
        const int per = T.R <= QUAD_VEC ? QUAD_BLOCK : 64;
        P.wgs = std::min(P.wgs, (long long)T.S * ((D.nbo + per - 1) / per));
    }
    P.rmax = rmax;
    return P;
}

}  // namespace

// The kernels' indices of octant nodes and of a face vector are 32-bit.
bool quad_indices_fit(const LevelHost& L) {
    long long N[3], noct = 1;
    for (int k = 0; k < 3; ++k) {
        N[k] = (long long)L.E[k] * L.n;
        noct *= (N[k] + 1) / 2;
    }
    return noct <= (1LL << 30) && 2 * (N[2] * N[1] + N[2] * N[0] + N[1] * N[0]) <= (1LL << 30);
}

// The widest tiles, whose padding may cost memory on a large grid (5 sources take the records of 16): beyond
// 8 GiB the records hold no more than a number of fields that follows the sources (in fours, at most 48).
QuadPlan quad_plan(const LevelHost& L, int nsrc) {
    const long long fields = nsrc < 4 ? nsrc : std::min(48, (nsrc + 3) / 4 * 4);
    for (int rmax : {32, 16}) {
        const QuadPlan P = quad_plan_width(L, nsrc, rmax, 1LL << 60);
        if (P.rec_len <= std::max(1LL << 30, L.ndof * fields)) return P;
    }
    return quad_plan_width(L, nsrc, QUAD_VEC, 1LL << 60);
}

// A plan whose records and partial sums fit in `capacity` doubles: the widest source tile that
// still leaves room for enough parts to give every launch about two work-groups a CU (or the most
// it can), narrower tiles meaning more passes over the octant.  rmax = 0: the mesh does not fit even
// with one source per pass and no split.
QuadPlan quad_plan_bounded(const LevelHost& L, int nsrc, long long capacity) {
    QuadPlan best{};
    for (int rmax : {32, 16, 4, 3, 2, 1}) {
        const QuadPlan P = quad_plan_width(L, nsrc, rmax, capacity);
        if (!P.rmax) {
            if (!best.nface) best = P;
            continue;
        }
        if (!best.rmax || P.wgs > best.wgs) best = P;
        if (P.wgs >= 512) return P;
    }
    return best;
}

void launch_quad_data(const LevelHost& L, const LevelDev<double>* dev, const double* nodes, const QuadPlan& P,
                      int nsrc, const double* f, const double* phi, const int* pi, const int* pj, double* rec,
                      double* part, double* g, hipStream_t s) {
    if (nsrc <= 0) return;
    const QuadDims D = quad_dims(L);
    const long long nfaces = 2 * ((long long)D.N[2] * D.N[1] + (long long)D.N[2] * D.N[0] + (long long)D.N[1] * D.N[0]);
    if (P.nface != nfaces || P.rmax < 1 || !quad_indices_fit(L))
        throw std::logic_error("quadrature plan does not fit the mesh");
    const double hmin = std::min({L.h[0], L.h[1], L.h[2]});
    const double drop2 = (1e-6 * hmin) * (1e-6 * hmin);
    const int nface = (int)nfaces;
    const double *xs = nodes, *ys = nodes + D.N[0], *zs = nodes + D.N[0] + D.N[1];
    for (int r0 = 0; r0 < nsrc;) {
        const int left = nsrc - r0;
        const QuadPass T = quad_pass(D, left, P.rmax, P.part_len, P.nface);
        const bool direct = T.S == 1, vec = T.R <= QUAD_VEC;
        if (8LL * D.noct * T.R > P.rec_len || (!direct && (!part || (long long)T.S * T.nr * nface > P.part_len)))
            throw std::logic_error("quadrature plan does not fit the mesh");
        const int per = vec ? QUAD_BLOCK : 64, ntb = (D.nbo + per - 1) / per;
        if ((long long)ntb * T.S >= (1LL << 31)) throw std::logic_error("quadrature grid too large");
        hipLaunchKernelGGL(k_quad_pack, dim3((unsigned)((D.noct + PACK_NODES - 1) / PACK_NODES)),
                           dim3(PACK_NODES * PACK_SRC), 0, s, dev, D, L.n, L.ndof, nsrc, r0, T.R, f, phi, pi, pj, rec);
        double* out = direct ? g + (long long)r0 * nface : part;
        switch (T.R) {
#define QUAD_CASE(RR, K, ...)                                                                                       \
    case RR:                                                                                                       \
        hipLaunchKernelGGL(K, dim3((unsigned)(ntb * T.S)), dim3(QUAD_BLOCK), 0, s, xs, ys, zs, D, nface, T.nper, ntb, \
                           drop2, rec, out __VA_ARGS__);                                                           \
        break;
            QUAD_CASE(1, k_quad<1>) QUAD_CASE(2, k_quad<2>) QUAD_CASE(3, k_quad<3>) QUAD_CASE(4, k_quad<4>)
            QUAD_CASE(16, k_quad_mfma<1>, , T.nr) QUAD_CASE(32, k_quad_mfma<2>, , T.nr)
#undef QUAD_CASE
            default: throw std::logic_error("no quadrature kernel for this tile");
        }
        hipLaunchKernelGGL(k_quad_combine, dim3((unsigned)((D.nbo + 255) / 256), (unsigned)T.nr), dim3(256), 0, s, out,
                           T.S, T.nr, D, nface, r0, dev, L.n, L.ndof, xs, ys, zs, drop2, f, phi, pi, pj, g);
        r0 += T.nr;
    }
}

}  // namespace dg
