// Field-side kernels for gfx950: Newmark right-hand side, PCG on a sliced-ELLPACK matrix
// (slice height 64 = one wavefront, coalesced column loads) with the nodal auxiliary-space
// preconditioner or with Jacobi, Faraday update and the conservation diagnostics.  Field
// vectors, residuals, dot products and the diagnostics are FP64; the PCG kernels are
// templated on their storage type, and the FP32 instances (matrix values, inverse
// diagonals and iteration vectors rounded to FP32, dot products and step lengths still
// FP64) run the inner passes of the mixed-precision solve.
//
// Grids are XCD-contiguous: the hardware hands workgroup b to XCD b % 8, so workgroup b
// walks the row blocks of the b % 8-th eighth of the rows, giving each XCD's L2 one
// contiguous stretch of rows and of the vector entries their columns mostly touch.
//
// But for the one-launch solves (k_cg_solve, k_pcg_solve, which pass values between running
// workgroups as tagged words), global dot products never communicate between workgroups
// inside a kernel: the once-per-solve reductions write one partial per workgroup that the next kernel sums
// (every workgroup, redundantly, in the same fixed order, so all reach the same bits);
// the iteration dots go through FP64-atomic slots that the next kernel sums the same way.
// Kernel boundaries give the visibility; no device-scope fences are issued.
#include <algorithm>

#include "fepic_internal.h"

namespace fepic {
namespace {

constexpr int kBlock = 256;
constexpr int kMaxGrid = 1024;  // 4 workgroups per CU on 256 CUs

struct RowGrid {
    int64_t nb;      // row blocks of kBlock rows
    int64_t per;     // row blocks per XCD
    int g;           // workgroups per XCD
    unsigned grid;   // 8 * g
};

inline RowGrid row_grid(int64_t n_rows, int max_grid = kMaxGrid) {
    RowGrid r;
    r.nb = (n_rows + kBlock - 1) / kBlock;
    r.per = (r.nb + 7) / 8;
    r.g = (int)std::min<int64_t>(r.per, max_grid / 8);
    if (r.g < 1) r.g = 1;
    r.grid = 8u * (unsigned)r.g;
    return r;
}

__device__ __forceinline__ int64_t rg_first(const RowGrid& rg) {
    return (int64_t)(blockIdx.x % 8) * rg.per + blockIdx.x / 8;
}
__device__ __forceinline__ int64_t rg_end(const RowGrid& rg) {
    const int64_t e = (int64_t)(blockIdx.x % 8 + 1) * rg.per;
    return e < rg.nb ? e : rg.nb;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// Block-wide sums of NV values over a block of BS threads; every thread receives the
// totals (summed in a fixed order).
template <int NV, int BS = kBlock>
__device__ __forceinline__ void block_sum_all(double v[NV]) {
    constexpr int NW = BS / 64;
    __shared__ double s[NV][NW];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const double x = wave_sum(v[j]);
        if (lane == 0) s[j][w] = x;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        double a = 0.0;
#pragma unroll
        for (int q = 0; q < NW; ++q) a += s[j][q];
        v[j] = a;
    }
    __syncthreads();
}

// Workgroup totals -> partial[j * gridDim.x + blockIdx.x].
template <int NV, int BS = kBlock>
__device__ __forceinline__ void write_partials(double v[NV], double* partial) {
    block_sum_all<NV, BS>(v);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int j = 0; j < NV; ++j) partial[(size_t)j * gridDim.x + blockIdx.x] = v[j];
    }
}

// Sum of the partials a previous kernel of n_src workgroups wrote (fixed order).
template <int NV, int BS = kBlock>
__device__ __forceinline__ void read_partials(const double* partial, int n_src, double tot[NV]) {
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        double a = 0.0;
        for (int b = threadIdx.x; b < n_src; b += BS) a += partial[(size_t)j * n_src + b];
        tot[j] = a;
    }
    block_sum_all<NV, BS>(tot);
}

// Sum over the row's slots of A(j,c) * f(c), four slots in flight at a time so the column
// and gather loads of a wavefront overlap (one thread per row, one wave per slice).
template <typename GatherFn>
__device__ __forceinline__ double sell_row(const int64_t* __restrict__ sp, const int32_t* __restrict__ col,
                                           const double* __restrict__ A, int64_t row, GatherFn f) {
    const int64_t sl = row >> 6;
    const int lane = (int)(row & 63);
    const int64_t k1 = sp[sl + 1];
    int64_t k = sp[sl] + lane;
    double acc0 = 0.0, acc1 = 0.0;
    for (; k + 3 * 64 < k1; k += 4 * 64) {
        const int c0 = col[k], c1 = col[k + 64], c2 = col[k + 128], c3 = col[k + 192];
        const double a0 = A[k], a1 = A[k + 64], a2 = A[k + 128], a3 = A[k + 192];
        const double u0 = f(c0), u1 = f(c1), u2 = f(c2), u3 = f(c3);
        acc0 += a0 * u0 + a2 * u2;
        acc1 += a1 * u1 + a3 * u3;
    }
    for (; k < k1; k += 64) acc0 += A[k] * f(col[k]);
    return acc0 + acc1;
}

__device__ __forceinline__ double sell_dot(const int64_t* __restrict__ sp, const int32_t* __restrict__ col,
                                           const double* __restrict__ val, const double* __restrict__ x,
                                           int64_t r) {
    const int64_t s = r >> 6;
    const int lane = (int)(r & 63);
    const int64_t b = sp[s], e = sp[s + 1];
    double acc = 0.0;
    for (int64_t k = b + lane; k < e; k += 64) acc += val[k] * x[col[k]];
    return acc;
}

__global__ __launch_bounds__(kBlock) void k_fill(double* x, int64_t n, double v) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) x[i] = v;
}

// Read-outs: the arrays' pieces (blockIdx.y) written in the caller's order straight into
// pinned host memory, whole cache lines at a time, so that neither a copy into pageable
// memory (16 GB/s here, against 55) nor the host's permutation is left.  Bound by the host's
// copy alongside: fields of 998k tets (35 MB) 5.7 -> 1.65 ms, 384k tets 2.0 -> 0.6.
__global__ __launch_bounds__(kBlock) void k_read_out(OutPieces pieces) {
    const OutPiece p = pieces.p[blockIdx.y];
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < p.n; i += (int64_t)gridDim.x * kBlock) {
        const int64_t j = p.perm ? p.perm[p.first + i] : p.first + i;
        if (p.kind == OUT_WORD)
            static_cast<unsigned long long*>(p.to)[i] = static_cast<const unsigned long long*>(p.src)[j];
        else if (p.kind == OUT_FLOAT)
            static_cast<double*>(p.to)[i] = (double)static_cast<const float*>(p.src)[j];
        else
            static_cast<int32_t*>(p.to)[i] = static_cast<const int32_t*>(p.src)[j];
    }
}

__global__ __launch_bounds__(kBlock) void k_axpby(double* y, const double* a, double alpha, const double* b,
                                                   double beta, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) y[i] = alpha * a[i] + beta * b[i];
}

// A = M + c S (+ cK K with absorbing faces); fixed (PEC) rows become identity rows.  The
// diagonal is slot 0 of every row (the host orders it first), so dinv = 1 / A(slot 0).
__global__ __launch_bounds__(kBlock) void k_scale_A(int64_t n_rows, const int64_t* __restrict__ sp,
                                                     const int32_t* __restrict__ col, const double* __restrict__ M,
                                                     const double* __restrict__ S, double* __restrict__ A,
                                                     double* __restrict__ dinv, const uint8_t* __restrict__ bmask,
                                                     double c, const double* __restrict__ K, double cK) {
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t s = r >> 6;
    const int lane = (int)(r & 63);
    if ((s << 6) >= n_rows) return;
    const int64_t b = sp[s], e = sp[s + 1];
    const bool real = r < n_rows;
    const bool bnd = real && bmask[r];
    for (int64_t k = b + lane; k < e; k += 64) {
        double a = M[k] + c * S[k];
        if (K) a += cK * K[k];
        if (bnd) a = (k == b + lane) ? 1.0 : 0.0;
        if (!real) a = 0.0;
        A[k] = a;
    }
    if (real) dinv[r] = 1.0 / A[b + lane];
}

__global__ __launch_bounds__(kBlock) void k_spmv(int64_t n_rows, const int64_t* __restrict__ sp,
                                                  const int32_t* __restrict__ col, const double* __restrict__ val,
                                                  const double* __restrict__ x, double* __restrict__ y) {
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if ((r >> 6) << 6 >= n_rows) return;
    const double v = sell_dot(sp, col, val, x, r);
    if (r < n_rows) y[r] = v;
}

// b = M (2 e - ep) - dt^2 S (c1 e + c2 ep) - (dg_new - dg_old), zero on fixed rows;
// partials of ||b||^2.  With absorbing faces (kAbc) also + K (kc1 e + kc2 ep), the damping
// terms of the Newmark recurrence.
template <bool kAbc>
__global__ __launch_bounds__(kBlock) void k_rhs(int64_t n_rows, RowGrid rg, const int64_t* __restrict__ sp,
                                                 const int32_t* __restrict__ col, const double* __restrict__ M,
                                                 const double* __restrict__ S, const double* __restrict__ e,
                                                 const double* __restrict__ ep, const double* __restrict__ dgn,
                                                 const double* __restrict__ dgo, const uint8_t* __restrict__ bmask,
                                                 double dt2, double c1, double c2, const double* __restrict__ K,
                                                 double kc1, double kc2, double* __restrict__ bvec,
                                                 double* __restrict__ partial) {
    double bb[1] = {0.0};
    for (int64_t lb = rg_first(rg), le = rg_end(rg); lb < le; lb += rg.g) {
        const int64_t r = lb * kBlock + threadIdx.x;
        if (((r >> 6) << 6) >= n_rows) continue;
        const int64_t s = r >> 6;
        const int lane = (int)(r & 63);
        const int64_t k0 = sp[s], k1 = sp[s + 1];
        double am = 0.0, as = 0.0, ak = 0.0;
        for (int64_t k = k0 + lane; k < k1; k += 64) {
            const int c = col[k];
            const double ec = e[c], epc = ep[c];
            am += M[k] * (2.0 * ec - epc);
            as += S[k] * (c1 * ec + c2 * epc);
            if constexpr (kAbc) ak += K[k] * (kc1 * ec + kc2 * epc);
        }
        if (r < n_rows) {
            double v = am - dt2 * as - (dgn[r] - dgo[r]);
            if constexpr (kAbc) v += ak;
            if (bmask[r]) v = 0.0;
            bvec[r] = v;
            bb[0] += v * v;
        }
    }
    write_partials<1>(bb, partial);
}

// The mixed (b, e) updates (FEPIC_FIELD_NM_MFEM, FEPIC_FIELD_BD_MFEM) with b^{n+1}
// eliminated: h = Mf (c1 b^n + c2 b^{n-1}) on face rows (Whitney-2 mass, SELL-64), then on
// edge rows
//   rhs = M (a0 e^n + a1 e^{n-1}) + dt^2 S (s0 e^n + s1 e^{n-1}) + dt sum_f C_fe h_f
//         - (g0 dG^{n+1} + g1 dG^n),
// C_fe from each edge's list of faces ((f << 1) | 1 for -1; -1 pads); wall rows 0.  The
// partials of ||rhs||^2 go where k_rhs puts them, for the solve that follows.
__global__ __launch_bounds__(kBlock) void k_face_spmv(int64_t n_faces, const int64_t* __restrict__ sp,
                                                       const int32_t* __restrict__ col, const double* __restrict__ val,
                                                       const double* __restrict__ b1, double c1,
                                                       const double* __restrict__ b2, double c2,
                                                       double* __restrict__ h) {
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (((r >> 6) << 6) >= n_faces) return;
    const int64_t sl = r >> 6;
    const int lane = (int)(r & 63);
    double acc = 0.0;
    for (int64_t k = sp[sl] + lane; k < sp[sl + 1]; k += 64) {
        const int c = col[k];
        acc += val[k] * (c1 * b1[c] + c2 * b2[c]);
    }
    if (r < n_faces) h[r] = acc;
}

struct MfemCoef {
    double a0, a1, s0, s1, g0, g1;
};

__global__ __launch_bounds__(kBlock) void k_mfem_rhs(int64_t n_rows, RowGrid rg, const int64_t* __restrict__ sp,
                                                      const int32_t* __restrict__ col, const double* __restrict__ M,
                                                      const double* __restrict__ S, const double* __restrict__ e,
                                                      const double* __restrict__ ep, const double* __restrict__ dgn,
                                                      const double* __restrict__ dgo, const uint8_t* __restrict__ bmask,
                                                      const int64_t* __restrict__ esp, const int32_t* __restrict__ einc,
                                                      const double* __restrict__ h, double dt, MfemCoef k,
                                                      double* __restrict__ bvec, double* __restrict__ partial) {
    double bb[1] = {0.0};
    for (int64_t lb = rg_first(rg), le = rg_end(rg); lb < le; lb += rg.g) {
        const int64_t r = lb * kBlock + threadIdx.x;
        if (((r >> 6) << 6) >= n_rows) continue;
        const int64_t s = r >> 6;
        const int lane = (int)(r & 63);
        double am = 0.0, as = 0.0, ac = 0.0;
        for (int64_t q = sp[s] + lane; q < sp[s + 1]; q += 64) {
            const int c = col[q];
            const double ec = e[c], epc = ep[c];
            am += M[q] * (k.a0 * ec + k.a1 * epc);
            as += S[q] * (k.s0 * ec + k.s1 * epc);
        }
        for (int64_t q = esp[s] + lane; q < esp[s + 1]; q += 64) {
            const int code = einc[q];
            if (code < 0) continue;
            const double hf = h[code >> 1];
            ac += (code & 1) ? -hf : hf;
        }
        if (r < n_rows) {
            double v = am + dt * dt * as + dt * ac - (k.g0 * dgn[r] + k.g1 * dgo[r]);
            if (bmask[r]) v = 0.0;
            bvec[r] = v;
            bb[0] += v * v;
        }
    }
    write_partials<1>(bb, partial);
}

// b^{n+1} = b_base - dt C (cn e^n + cm e^{n-1} + cp e^{n+1}) (NM: b_base = b^{n-1},
// coefficients 1, 1/2, 1/2; BD: b_base = b^n, 0, 0, 1).
__global__ __launch_bounds__(kBlock) void k_mfem_faraday(int64_t n_faces, const int32_t* __restrict__ fe,
                                                          const double* __restrict__ b_base,
                                                          const double* __restrict__ e_n,
                                                          const double* __restrict__ e_nm1,
                                                          const double* __restrict__ e_np1, double dt, double cn,
                                                          double cm, double cp, double* __restrict__ b_new) {
    const int64_t f = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (f >= n_faces) return;
    double v = 0.0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int a = fe[3 * f + j];
        const double ea = cn * e_n[a] + cm * e_nm1[a] + cp * e_np1[a];
        v += j == 2 ? -ea : ea;
    }
    b_new[f] = b_base[f] - dt * v;
}

__global__ __launch_bounds__(kBlock) void k_warm(int mode, int64_t n, const double* __restrict__ e,
                                                  const double* __restrict__ ep, const double* __restrict__ ep2,
                                                  double* __restrict__ x) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    double v = e[i];
    if (mode == FEPIC_WS_EXTRAP1) v = 2.0 * e[i] - ep[i];
    if (mode == FEPIC_WS_EXTRAP2) v = 3.0 * e[i] - 3.0 * ep[i] + ep2[i];
    x[i] = v;
}

// Jacobi-preconditioned CG in the single-reduction form of Chronopoulos and Gear (1989):
// with u = D^-1 r and w = A u kept by recurrence, one iteration needs the three dots
// (r,u), (u,w), (r,r) of the previous iterate only, so it is one kernel:
//   beta_i  = g_i / g_{i-1},   alpha_i = g_i / (d_i - beta_i g_i / alpha_{i-1})
//   p = u + beta p,  s = w + beta s,  x += alpha p,  r' = r - alpha s,  u' = D^-1 r',
//   w' = A u' (the neighbours' u' formed on the fly from the previous r, w, s),
//   g_{i+1} = (r',u'), d_{i+1} = (u',w'), ||r'||^2.
// The kernel keeps r, w and s scaled by D^-1 (R = D^-1 r, W = D^-1 w, S = D^-1 s, D =
// diag A) so a neighbour's u' = R - alpha (W + beta S) needs three of its values; they
// are stored interleaved with the row's own p (CgVec, 32 bytes per row) so the three
// come from one sector.  The interleaved state is double buffered (neighbours read the
// previous values); x is touched by its own row only.

// Iteration partials: the three dots of each iteration are added with FP64 atomics into
// kCgSlots slots per value (workgroup b -> slot b mod kCgSlots), in three rotating
// buffers: iteration i reads buffer i mod 3 (filled by the previous kernel), adds into
// buffer (i + 1) mod 3 (cleared by the previous kernel) and clears buffer (i + 2) mod 3
// (read by the previous kernel).  Reading 3 x 64 values instead of one partial per
// workgroup lets the iteration kernel run one workgroup per row block at any size.
constexpr int kCgSlots = 64;
__device__ __forceinline__ double* cg_buf(double* base, int k) { return base + (size_t)(k % 3) * 3 * kCgSlots; }

// Workgroup totals v (already summed over the block) added into buffer slots.
__device__ __forceinline__ void cg_add(double* buf, const double v[3]) {
    if (threadIdx.x == 0) {
        const int s = blockIdx.x & (kCgSlots - 1);
#pragma unroll
        for (int j = 0; j < 3; ++j) unsafeAtomicAdd(buf + j * kCgSlots + s, v[j]);
    }
}

// ||b||^2 from the right-hand side's partials; R = D^-1 (b - A x); W = S = P = 0; clears
// iteration buffers 0 and 1.
__global__ __launch_bounds__(kBlock) void k_cg_init_a(int64_t n_rows, RowGrid rg, const int64_t* __restrict__ sp,
                                                       const int32_t* __restrict__ col, const double* __restrict__ A,
                                                       const double* __restrict__ dinv, const double* __restrict__ b,
                                                       const double* __restrict__ x, CgVec* __restrict__ V,
                                                       const double* __restrict__ part_rhs, int n_rhs_wg,
                                                       double* cg_slots, CgScalars* sc, double tol) {
    double bb[1];
    read_partials<1>(part_rhs, n_rhs_wg, bb);
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            sc->bb = bb[0];
            sc->tol2_bb = tol * tol * bb[0];
            sc->converged = 0;
            sc->gave_up = 0;
        }
        for (int k = threadIdx.x; k < 2 * 3 * kCgSlots; k += kBlock) cg_slots[k] = 0.0;
    }
    for (int64_t lb = rg_first(rg), le = rg_end(rg); lb < le; lb += rg.g) {
        const int64_t row = lb * kBlock + threadIdx.x;
        if (((row >> 6) << 6) >= n_rows) continue;
        const double ax = sell_row(sp, col, A, row, [&](int c) { return x[c]; });
        if (row < n_rows) {
            double2* o = reinterpret_cast<double2*>(V + row);
            o[0] = make_double2(dinv[row] * (b[row] - ax), 0.0);
            o[1] = make_double2(0.0, 0.0);
        }
    }
}

// W = D^-1 A u with u = R (only R is gathered); partials of (r,u), (u,w), (r,r).
__global__ __launch_bounds__(kBlock) void k_cg_init_b(int64_t n_rows, RowGrid rg, const int64_t* __restrict__ sp,
                                                       const int32_t* __restrict__ col, const double* __restrict__ A,
                                                       const double* __restrict__ dinv, CgVec* __restrict__ V,
                                                       double* __restrict__ cg_slots) {
    double v[3] = {0.0, 0.0, 0.0};
    for (int64_t lb = rg_first(rg), le = rg_end(rg); lb < le; lb += rg.g) {
        const int64_t row = lb * kBlock + threadIdx.x;
        if (((row >> 6) << 6) >= n_rows) continue;
        const double acc = sell_row(sp, col, A, row, [&](int c) { return V[c].R; });
        if (row < n_rows) {
            const double dj = dinv[row], uv = V[row].R, rv = uv / dj;
            V[row].W = dj * acc;
            v[0] += rv * uv;
            v[1] += uv * acc;
            v[2] += rv * rv;
        }
    }
    block_sum_all<3>(v);
    cg_add(cg_buf(cg_slots, 0), v);
}

// ------------------------------------------------------------------------------------
// PCG with the nodal auxiliary-space preconditioner of Hiptmair and Xu (2007), additive,
// one Jacobi step in each space:  B r = D^-1 r + G D_G^-1 G^T r + Pi D_Pi^-1 Pi^T r,
// D = diag A, D_G = diag G^T A G, D_Pi = diag Pi^T A Pi, G the discrete gradient and Pi the
// vector nodal interpolation on interior edges and nodes, plus the same two corrections
// for piecewise-constant nodal fields on aggregates of 8, 64 (within a node slice) and
// 512, 4096, 32768 (far levels) Morton-consecutive nodes.  The slow components of
// Jacobi-PCG on the Newmark system are gradients (the kernel of S) and smooth curl
// fields; the nodal spaces reach both.  Plain (Hestenes-Stiefel) recurrences; an
// iteration is three kernels (four with far levels), because z = B r needs the nodal sums
// of the new residual before any edge can form it:
//   k_pcg_q(i):      beta = g_i / g_{i-1};  p = z + beta p;  q = A p (the neighbours' p
//                    formed on the fly from their gathered (z, p) pair);  dot (p, q)
//   k_pcg_nodes(i):  alpha = g_i / (p, q);  per interior node, G^T r' and Pi^T r' over its
//                    edges, r' = r - alpha q, scaled by D_G^-1 and D_Pi^-1, plus the
//                    aggregate levels of the node's slice; the finest far level's sums
//                    by atomics
//   k_pcg_fold(i):   with far levels, the coarser far levels' sums from the finest
//                    level's, then each node's Y += its far aggregates' sums times their
//                    scales (once per node, not at both ends of every edge)
//   k_pcg_update(i): p again (same operands, same bits);  x += alpha p;  r = r';
//                    z = D^-1 r + G y + Pi v (all levels);  dots (r, z), (r, r)
// (Meshes of up to 262k rows do all of this in one launch per solve, k_pcg_solve.)
// Every kernel issues its loads before it sums the previous kernel's slots.  Reductions
// use the iteration slots in four rotating buffers: reduction k goes to buffer k mod 4;
// iteration i adds (p, q) as reduction 2i and (r, z), (r, r) as reduction 2i + 1; the
// start's dots are reduction -1.  k_pcg_nodes(i) clears buffer 2i + 1 and
// k_pcg_update(i) buffer 2i + 2, each after that buffer's last reader and before its next
// writer.
__device__ __forceinline__ double* red_buf(double* base, int k) {
    return base + (size_t)(((k % 4) + 4) % 4) * 3 * kCgSlots;
}

__device__ __forceinline__ void clear_buf(double* buf) {
    for (int k = threadIdx.x; k < 3 * kCgSlots; k += kBlock) buf[k] = 0.0;
}

__device__ __forceinline__ double3 edge_vec(const AuxSpace& g, int64_t e) {
    const EdgeVec t = g.th[e];
    return make_double3((double)(float)t.x, (double)(float)t.y, (double)(float)t.z);
}

// Per node: D_G^-1 and D_Pi^-1 from the rows of A.  The pair (e, f) of the node's edges
// contributes s_e A_ef s_f to diag G^T A G (s = +1 at an edge's head, -1 at its tail) and
// th_e,d A_ef th_f,d to component d of diag Pi^T A Pi; f runs over row e's stored columns
// and counts when the node is one of its ends.
__global__ __launch_bounds__(kBlock) void k_aux_scale(AuxSpace g, const int64_t* __restrict__ sp,
                                                       const int32_t* __restrict__ col, const double* __restrict__ A) {
    const int64_t n = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (n >= g.n_aux) return;
    const int64_t sl = n >> 6;
    const int lane = (int)(n & 63);
    double dg = 0.0, dp0 = 0.0, dp1 = 0.0, dp2 = 0.0;
    for (int64_t k = g.sp[sl] + lane; k < g.sp[sl + 1]; k += 64) {
        const int32_t c = g.inc[k];
        if (c == kAuxPad) continue;
        const int32_t e = c >= 0 ? c : ~c;
        const double se = c >= 0 ? 1.0 : -1.0;
        const double3 te = edge_vec(g, e);
        const int64_t esl = e >> 6;
        const int el = e & 63;
        for (int64_t kk = sp[esl] + el; kk < sp[esl + 1]; kk += 64) {
            const int32_t f = col[kk];
            const int2 ef = g.ends[f];
            const double sf = ef.y == n ? 1.0 : (ef.x == n ? -1.0 : 0.0);
            if (sf == 0.0) continue;
            const double a = A[kk];
            const double3 tf = edge_vec(g, f);
            dg += se * a * sf;
            dp0 += (double)te.x * a * (double)tf.x;
            dp1 += (double)te.y * a * (double)tf.y;
            dp2 += (double)te.z * a * (double)tf.z;
        }
    }
    g.scale[n] = make_double4(dg > 0.0 ? 1.0 / dg : 0.0, dp0 > 0.0 ? 1.0 / dp0 : 0.0, dp1 > 0.0 ? 1.0 / dp1 : 0.0,
                              dp2 > 0.0 ? 1.0 / dp2 : 0.0);
}

// Diagonals of the aggregate levels: for aggregate a (aux nodes [a L, (a + 1) L)) the
// G-level basis vector is phi_e = (head of e in a) - (tail of e in a) and the Pi-level one
// psi_e = th_e ((tail in a) + (head in a)); diag = phi^T A phi and psi_d^T A psi_d.  Each
// node adds the terms of its incident edges, an edge with both ends in the aggregate from
// its tail only, into the aggregate's accumulator (zeroed before).
template <int kLog>
__device__ __forceinline__ void coarse_terms(const AuxSpace& g, const int64_t* __restrict__ sp,
                                             const int32_t* __restrict__ col, const double* __restrict__ A,
                                             int64_t n, double out[4]) {
    const int64_t agg = n >> kLog;
    auto in_agg = [&](int32_t k) { return k < g.n_aux && ((int64_t)k >> kLog) == agg; };
    const int64_t sl = n >> 6;
    const int lane = (int)(n & 63);
    double dg = 0.0, dp0 = 0.0, dp1 = 0.0, dp2 = 0.0;
    for (int64_t k = g.sp[sl] + lane; k < g.sp[sl + 1]; k += 64) {
        const int32_t c = g.inc[k];
        if (c == kAuxPad) continue;
        const int32_t e = c >= 0 ? c : ~c;
        const int2 ee = g.ends[e];
        const bool t_in = in_agg(ee.x), h_in = in_agg(ee.y);
        if (c >= 0 && t_in) continue;   // head end of an edge inside the aggregate: its tail counts it
        const double phe = (h_in ? 1.0 : 0.0) - (t_in ? 1.0 : 0.0);
        const double pse = (t_in ? 1.0 : 0.0) + (h_in ? 1.0 : 0.0);
        const double3 te = edge_vec(g, e);
        const int64_t esl = e >> 6;
        const int el = e & 63;
        double rg = 0.0, r0 = 0.0, r1 = 0.0, r2 = 0.0;   // (A phi)_e, (A psi_d)_e
        for (int64_t kk = sp[esl] + el; kk < sp[esl + 1]; kk += 64) {
            const int32_t f = col[kk];
            const int2 ef = g.ends[f];
            const bool ft = in_agg(ef.x), fh = in_agg(ef.y);
            if (!ft && !fh) continue;
            const double a = A[kk];
            const double3 tf = edge_vec(g, f);
            const double phf = (fh ? 1.0 : 0.0) - (ft ? 1.0 : 0.0);
            const double psf = (ft ? 1.0 : 0.0) + (fh ? 1.0 : 0.0);
            rg += a * phf;
            r0 += a * psf * (double)tf.x;
            r1 += a * psf * (double)tf.y;
            r2 += a * psf * (double)tf.z;
        }
        dg += phe * rg;
        dp0 += pse * (double)te.x * r0;
        dp1 += pse * (double)te.y * r1;
        dp2 += pse * (double)te.z * r2;
    }
    out[0] = dg;
    out[1] = dp0;
    out[2] = dp1;
    out[3] = dp2;
}

__device__ __forceinline__ void add4(double4* acc, const double v[4]) {
    double* o = reinterpret_cast<double*>(acc);
#pragma unroll
    for (int k = 0; k < 4; ++k) unsafeAtomicAdd(o + k, v[k]);
}

// Aggregates of 8 and 64 nodes take one atomic per node; the far levels (whole
// workgroups of consecutive nodes per aggregate) one per workgroup.
__global__ __launch_bounds__(kBlock) void k_aux_coarse(AuxSpace g, const int64_t* __restrict__ sp,
                                                        const int32_t* __restrict__ col, const double* __restrict__ A) {
    static_assert(aux_far_log(0) >= 8, "a far aggregate holds whole workgroups");
    const int64_t n = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const bool real = n < g.n_aux;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (real) {
        coarse_terms<3>(g, sp, col, A, n, v);
        add4(g.scale8 + (n >> 3), v);
        coarse_terms<6>(g, sp, col, A, n, v);
        add4(g.scale64 + (n >> 6), v);
    }
#pragma unroll
    for (int L = 0; L < kAuxFarLevels; ++L) {
        if (real) {
            static_assert(kAuxFarLevels == 3, "one coarse_terms instance per far level");
            if (L == 0) coarse_terms<aux_far_log(0)>(g, sp, col, A, n, v);
            else if (L == 1) coarse_terms<aux_far_log(1)>(g, sp, col, A, n, v);
            else coarse_terms<aux_far_log(2)>(g, sp, col, A, n, v);
        } else {
            v[0] = v[1] = v[2] = v[3] = 0.0;
        }
        block_sum_all<4>(v);
        if (threadIdx.x == 0) add4(g.far_scale[L] + (((int64_t)blockIdx.x * kBlock) >> aux_far_log(L)), v);
    }
}

// diag -> 1 / diag in place (0 where the diagonal is not positive).
__global__ __launch_bounds__(kBlock) void k_invert_pos(double* v, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) v[i] = v[i] > 0.0 ? 1.0 / v[i] : 0.0;
}

// Zeroes the finest far level's accumulators, the only ones the node pass adds into (one
// workgroup).
__device__ __forceinline__ void clear_far(const AuxSpace& g) {
    if (g.n_far < 1) return;
    const int64_t nf = (g.n_aux + (1ll << aux_far_log(0)) - 1) >> aux_far_log(0);
    double* a = reinterpret_cast<double*>(g.far_acc);
    for (int64_t k = threadIdx.x; k < 4 * nf; k += kBlock) a[8 * k] = 0.0;
}

// The accumulator of component comp of the finest far level's aggregate a: one 64-byte
// line each.
__device__ __forceinline__ double* far_line(const AuxSpace& g, int64_t a, int comp) {
    return reinterpret_cast<double*>(g.far_acc) + 8 * (4 * a + comp);
}

// Storage of the iteration: FP64, or FP32 for the inner solves of the mixed-precision
// form (scalars and dot products stay FP64 either way).
template <typename S>
struct Vec;
template <>
struct Vec<double> {
    using t2 = double2;
    using t3 = double3;
    using t4 = double4;
    static __device__ __forceinline__ double2 two(double a, double b) { return make_double2(a, b); }
    static __device__ __forceinline__ double4 four(double a, double b, double c, double d) {
        return make_double4(a, b, c, d);
    }
};
template <>
struct Vec<float> {
    using t2 = float2;
    using t3 = float3;
    using t4 = float4;
    static __device__ __forceinline__ float2 two(float a, float b) { return make_float2(a, b); }
    static __device__ __forceinline__ float4 four(float a, float b, float c, float d) {
        return make_float4(a, b, c, d);
    }
};

// The FP64 or the FP32 copy of an auxiliary-space array.
template <typename S, typename D, typename F>
__device__ __forceinline__ auto pick(D d, F f) {
    if constexpr (sizeof(S) == 8)
        return d;
    else
        return f;
}

template <typename S>
__device__ __forceinline__ typename Vec<S>::t3 edge_vec_t(const AuxSpace& g, int64_t e) {
    const EdgeVec t = g.th[e];
    typename Vec<S>::t3 v;
    v.x = (S)(float)t.x;
    v.y = (S)(float)t.y;
    v.z = (S)(float)t.z;
    return v;
}

// Sum over the wave by DPP moves (row shifts, then the rows' totals carried across), the
// same bits in every lane: VALU moves, where shuffles would be LDS permutes.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ double dpp_add(double v) {
#pragma clang fp contract(off)
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), kCtrl, kRowMask, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), kCtrl, kRowMask, 0xf, true);
    return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_total(double v) {
    v = dpp_add<0x111, 0xf>(v);   // row_shr:1
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);   // row_bcast:15
    v = dpp_add<0x143, 0xc>(v);   // row_bcast:31
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                            __builtin_amdgcn_readlane(__double2loint(v), 63));
}

// A reduction's kCgSlots slots, one per lane: every wave loads and sums them itself (the
// same bits everywhere), which costs a few cache hits and no barrier.  With the recurrence's
// scalars loaded at the top of each kernel rather than after that sum, and one barrier per
// workgroup total, an iteration's three or four kernels lost 1.2-1.6 us in all: 41k tets,
// FP64, 14.5 -> 13.3 us; beam, FP32, 18.2 -> 17.1; 998k tets 52.1 -> 50.6.
template <int NV>
__device__ __forceinline__ void slot_load_wave(const double* buf, double t[NV]) {
    static_assert(kCgSlots == 64, "one slot per lane");
#pragma unroll
    for (int j = 0; j < NV; ++j) t[j] = buf[j * kCgSlots + (threadIdx.x & 63)];
}

// Workgroup totals of v into the workgroup's slots (R threads; one barrier).
template <int NV, int R>
__device__ __forceinline__ void block_slot_add(const double v[NV], double* buf) {
    __shared__ double s[NV][R / 64];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const double w = wave_total(v[j]);
        if ((threadIdx.x & 63) == 0) s[j][threadIdx.x >> 6] = w;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        double a = 0.0;
#pragma unroll
        for (int q = 0; q < R / 64; ++q) a += s[threadIdx.x][q];
        unsafeAtomicAdd(buf + threadIdx.x * kCgSlots + (blockIdx.x & (kCgSlots - 1)), a);
    }
}

// One row's slice of the matrix, its first 2 kPairs slots in registers (issued before the
// staged vector is known): all of a row on the workloads' meshes (at most 19 slots).
template <typename S>
struct BlockRow {
    static constexpr int kPairs = 10;
    S a[2 * kPairs];
    uint32_t c[kPairs];
    int64_t k0;   // the lane's first slot
    int w;        // slots per row of the slice (0 past the matrix)

    // slots 2 j and 2 j + 1 (the second zero past the width)
    __device__ __forceinline__ void pair(const BlockCols& bc, const S* __restrict__ A, int j, S& a0, S& a1,
                                         uint32_t& cc) const {
        const int lane = threadIdx.x & 63;
        if (2 * j + 1 < w) {
            const int64_t k = k0 + 128 * j + 2 * lane;
            cc = *reinterpret_cast<const uint32_t*>(bc.lcol + k);
            if constexpr (sizeof(S) == 4) {   // the FP32 copy has the pair layout
                const float2 v = *reinterpret_cast<const float2*>(A + k);
                a0 = v.x;
                a1 = v.y;
            } else {
                a0 = A[k0 + 128 * j + lane];
                a1 = A[k0 + 128 * j + 64 + lane];
            }
        } else {
            cc = bc.lcol[k0 + 128 * j + lane];
            a0 = A[k0 + 128 * j + lane];
            a1 = S(0);
        }
    }
    __device__ __forceinline__ void load(const BlockCols& bc, int64_t slice, const int64_t* __restrict__ sp,
                                         const S* __restrict__ A) {
        const int sl = __builtin_amdgcn_readfirstlane((int)slice);   // wave-uniform: scalar loads
        k0 = 0;
        w = 0;
        if (sl < bc.n_slices) {
            k0 = sp[sl];
            w = (int)((sp[sl + 1] - k0) >> 6);
        }
#pragma unroll
        for (int j = 0; j < kPairs; ++j)
            if (2 * j < w) pair(bc, A, j, a[2 * j], a[2 * j + 1], c[j]);
    }
    // sum over the row of A f(local column)
    template <typename F>
    __device__ __forceinline__ S dot(const BlockCols& bc, const S* __restrict__ A, F f) const {
        S s0 = S(0), s1 = S(0);
#pragma unroll
        for (int j = 0; j < kPairs; ++j)
            if (2 * j < w) {
                s0 = fma(a[2 * j], f(c[j] & 0xffffu), s0);
                s1 = fma(a[2 * j + 1], f(c[j] >> 16), s1);
            }
        for (int j = kPairs; 2 * j < w; ++j) {
            S a0, a1;
            uint32_t cc;
            pair(bc, A, j, a0, a1, cc);
            s0 = fma(a0, f(cc & 0xffffu), s0);
            s1 = fma(a1, f(cc >> 16), s1);
        }
        return s0 + s1;
    }
    // the same by the 32-bit columns (a block whose halo exceeds kHaloMax)
    template <typename F>
    __device__ __forceinline__ S dot_wide(const int32_t* __restrict__ col, const S* __restrict__ A, F f) const {
        const int lane = threadIdx.x & 63;
        S s = S(0);
#pragma unroll 4
        for (int k = 0; k < w; ++k) {
            int64_t ka = k0 + 64 * k + lane;
            if (sizeof(S) == 4 && (k | 1) < w) ka = k0 + 128 * (k >> 1) + 2 * lane + (k & 1);
            s += A[ka] * f(col[k0 + 64 * k + lane]);
        }
        return s;
    }
};

// Halo columns a thread stages from registers (1,024 per block; more in a loop).
constexpr int kHaloRegs = 1024 / kBlockRows;

__device__ __forceinline__ void halo_ids(const BlockCols& bc, int64_t b, int h[kHaloRegs]) {
#pragma unroll
    for (int k = 0; k < kHaloRegs; ++k)
        if (k * kBlockRows < bc.stride) h[k] = bc.halo[b * bc.stride + k * kBlockRows + threadIdx.x];
}

// One workgroup per row block.  The halo (distinct columns outside the block) is found by
// inserting the block's columns into an LDS hash table, then sorted, so that its gathers run
// through memory in order; with kFill the lists and each slot's 16-bit index (own rows
// first, then the halo position, by binary search) are written, otherwise the counts only.
// A block of more than kHaloMax halo columns gets cnt -1 and no indices.  Every loop is
// bounded: the table has twice kHaloMax slots, inserts stop once kHaloMax is passed (at most
// one more per thread is under way), and a probe visits each slot once.
template <bool kFill>
__global__ __launch_bounds__(kBlock) void k_block_cols(BlockCols g, const int64_t* __restrict__ sp,
                                                        const int32_t* __restrict__ col, int32_t* __restrict__ cnt,
                                                        int32_t* __restrict__ halo, uint16_t* __restrict__ lcol) {
    constexpr int kTable = 2 * kHaloMax;
    __shared__ int s_key[kTable];
    __shared__ int s_list[kHaloMax];
    __shared__ int s_n, s_m;
    const int64_t b = blockIdx.x, r0 = b * kBlockRows, r1 = r0 + kBlockRows;
    const int64_t sl0 = r0 >> 6, sl1 = min((int64_t)(r1 >> 6), g.n_slices);
    const int64_t k0 = sp[sl0], k1 = sp[sl1];
    for (int k = threadIdx.x; k < kTable; k += kBlock) s_key[k] = -1;
    if (threadIdx.x == 0) s_n = s_m = 0;
    __syncthreads();
    for (int64_t k = k0 + threadIdx.x; k < k1; k += kBlock) {
        const int c = col[k];
        if (c >= r0 && c < r1) continue;
        unsigned h = ((unsigned)c * 2654435761u) >> (32 - 13);
        static_assert(kTable == 1 << 13, "hash width");
        for (int p = 0; p < kTable; ++p) {
            const int old = __hip_atomic_load(s_key + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (old == c) break;
            if (old == -1) {
                if (__hip_atomic_load(&s_n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > kHaloMax) break;
                const int was = atomicCAS(s_key + h, -1, c);
                if (was == -1) atomicAdd(&s_n, 1);
                if (was == -1 || was == c) break;
            }
            h = (h + 1) & (kTable - 1);
        }
    }
    __syncthreads();
    const int n = s_n;
    if (!kFill) {
        if (threadIdx.x == 0) cnt[b] = n > kHaloMax ? -1 : n;
        return;
    }
    if (n > kHaloMax) {
        for (int k = threadIdx.x; k < g.stride; k += kBlock) halo[b * g.stride + k] = (int32_t)r0;
        return;
    }
    int n2 = 1;
    while (n2 < n) n2 <<= 1;
    for (int k = threadIdx.x; k < kTable; k += kBlock)
        if (s_key[k] >= 0) s_list[atomicAdd(&s_m, 1)] = s_key[k];
    __syncthreads();
    for (int k = n + threadIdx.x; k < n2; k += kBlock) s_list[k] = INT32_MAX;
    __syncthreads();
    for (int sz = 2; sz <= n2; sz <<= 1)   // bitonic sort
        for (int d = sz >> 1; d > 0; d >>= 1) {
            for (int k = threadIdx.x; k < n2 / 2; k += kBlock) {
                const int i = 2 * k - (k & (d - 1)), j = i + d;
                const int x = s_list[i], y = s_list[j];
                if ((x > y) == ((i & sz) == 0)) {
                    s_list[i] = y;
                    s_list[j] = x;
                }
            }
            __syncthreads();
        }
    for (int k = threadIdx.x; k < g.stride; k += kBlock) halo[b * g.stride + k] = k < n ? s_list[k] : (int32_t)r0;
    for (int64_t sl = sl0; sl < sl1; ++sl) {
        const int64_t base = sp[sl];
        const int w = (int)((sp[sl + 1] - base) >> 6);
        for (int e = threadIdx.x; e < 64 * w; e += kBlock) {
            const int k = e >> 6, lane = e & 63, c = col[base + e];
            int idx;
            if (c >= r0 && c < r1) {
                idx = (int)(c - r0);
            } else {
                int lo = 0, hi = n - 1;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (s_list[mid] < c) lo = mid + 1;
                    else hi = mid;
                }
                idx = kBlockRows + lo;
            }
            lcol[base + ((k | 1) < w ? 128 * (k >> 1) + 2 * lane + (k & 1) : e)] = (uint16_t)idx;
        }
    }
}

// The FP32 values of a SELL-64 matrix in the pair layout (one wave per slice).
__global__ __launch_bounds__(kBlock) void k_pack_f32(int64_t n_slices, const int64_t* __restrict__ sp,
                                                      const double* __restrict__ A, float* __restrict__ A32) {
    const int64_t sl = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (sl >= n_slices) return;
    const int lane = threadIdx.x & 63;
    const int64_t k0 = sp[sl];
    const int w = (int)((sp[sl + 1] - k0) >> 6);
    int k = 0;
    for (; k + 1 < w; k += 2)
        *reinterpret_cast<float2*>(A32 + k0 + 64 * k + 2 * lane) =
            make_float2((float)A[k0 + 64 * k + lane], (float)A[k0 + 64 * k + 64 + lane]);
    if (k < w) A32[k0 + 64 * k + lane] = (float)A[k0 + 64 * k + lane];
}

// What the Jacobi-PCG kernels compute alike.  Products and sums are kept apart, and the
// multiply-adds of the recurrences written out, because which of them a compiler fuses is its
// choice in each kernel, and k_cg_iter<true> has to give k_cg_solve's bits.
struct CgStep {
    double alpha, beta;
    int conv;   // 1: done, 2: breakdown
};
__device__ __forceinline__ CgStep cg_step(int i, double g, double d, double rr, double gam_old, double alpha_old,
                                          double tol2_bb, double bb) {
#pragma clang fp contract(off)
    const bool done = !(rr > tol2_bb) || bb == 0.0;
    const double beta = (i == 0) ? 0.0 : g / gam_old;
    const double alpha = (i == 0) ? g / d : g / (d - beta * g / alpha_old);
    const bool bad = !done && !(alpha > 0.0 && alpha < INFINITY && beta >= 0.0 && beta < INFINITY);
    return {alpha, beta, done ? 1 : (bad ? 2 : 0)};
}
// (r, u), (u, w) and (r, r) of a row, D^-1 r = u.
__device__ __forceinline__ void cg_dots(double u, double acc, double diag, double v[3]) {
#pragma clang fp contract(off)
    const double rn = u * diag;
    v[0] = rn * u;
    v[1] = u * acc;
    v[2] = rn * rn;
}
// The waves' sums of v, and their sum.
template <int NV, int NW>
__device__ __forceinline__ void sum_waves(const double v[NV], double (*s)[NW]) {
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const double a = wave_total(v[j]);
        if ((threadIdx.x & 63) == 0) s[j][threadIdx.x >> 6] = a;
    }
}
template <int NW>
__device__ __forceinline__ double over_waves(const double* s) {
    double a = 0.0;
#pragma unroll
    for (int q = 0; q < NW; ++q) a += s[q];
    return a;
}

// One Jacobi-PCG iteration per row block.  The neighbours'
// u' = R - alpha (W + beta S) are staged in LDS like the auxiliary-space product's p, one
// value per column instead of three gathered values per stored slot; a row's diagonal is its
// slot 0.  Bound by HBM on large meshes (998k tets: 92.8 -> 55.4 us), by the chain of
// dependent loads on small ones, where the six-at-a-time gathers took up to twelve round
// trips: beam 19.7 -> 13.1 us, 29k tets 8.2 -> 6.9, 1.3k tets 7.6 -> 5.1; deterministic, 13k
// tets, 10.6 -> 6.0.
// kTwin false: meshes past k_cg_solve's limits (more row blocks than CUs, or a halo too long
// for its registers); the dots go into slots, and in the deterministic mode a workgroup takes
// every rg.g-th block, so that each slot takes a single add.
// kTwin true: meshes within them, where that solve was given up, refused or switched off.  Its
// arithmetic to the bit, so that a deterministic step is the same whichever of the two made
// it: the workgroups' partials one per thread, summed in its order (part: two buffers of
// [3][kBlockRows]), and no update past n_max.
template <bool kTwin>
__global__ __launch_bounds__(kBlockRows) void k_cg_iter(int64_t n_rows, RowGrid rg, int i, int n_max,
                                                         const int64_t* __restrict__ sp,
                                                         const int32_t* __restrict__ col, BlockCols bc,
                                                         const double* __restrict__ A, double* __restrict__ x,
                                                         const CgVec* __restrict__ V, CgVec* __restrict__ V_new,
                                                         double* __restrict__ cg_slots, double* __restrict__ part,
                                                         CgScalars* sc) {
    extern __shared__ double s_u[];
    constexpr int R = kBlockRows, H = kHaloRegs, NW = R / 64;
    __shared__ double s_dot[kTwin ? 3 : 1][NW];
    // The converged flag, the previous kernel's dot slots and this workgroup's first block
    // are all in flight together; the flag (the same for every thread) is checked before
    // any write, so a launch after convergence changes nothing.
    const int conv = sc->converged;
    const double tol2_bb = sc->tol2_bb, bb = sc->bb, gam_old = sc->gam[(i + 1) & 1], alpha_old = sc->alpha[(i + 1) & 1];
    double t[3];
    if (!kTwin || i == 0) {
        slot_load_wave<3>(kTwin ? cg_slots : cg_buf(cg_slots, i), t);
    } else {
#pragma unroll
        for (int j = 0; j < 3; ++j)
            t[j] = threadIdx.x < bc.nb ? part[(3 * (i & 1) + j) * R + threadIdx.x] : 0.0;
    }
    int64_t b = rg_first(rg);
    const int64_t le = rg_end(rg);
    if (b >= le) return;   // the whole workgroup
    BlockRow<double> P;
    double2 own_rw, own_sp, rw[H];
    double own_x, hs[H];
    int cnt;
    auto load = [&]() {
        const int64_t row = b * R + threadIdx.x, r = row < n_rows ? row : 0;
        P.load(bc, b * (R / 64) + (threadIdx.x >> 6), sp, A);
        cnt = bc.cnt[b];
        int h[H];
        halo_ids(bc, b, h);
        const double2* o = reinterpret_cast<const double2*>(V + r);
        own_rw = o[0];
        own_sp = o[1];
        own_x = x[r];
#pragma unroll
        for (int k = 0; k < H; ++k)
            if (k * R < bc.stride) {
                rw[k] = *reinterpret_cast<const double2*>(V + h[k]);
                hs[k] = V[h[k]].S;
            }
    };
    load();
    double g, d, rr;
    if (!kTwin || i == 0) {
        g = wave_total(t[0]);
        d = wave_total(t[1]);
        rr = wave_total(t[2]);
    } else {
        // by all waves, also one that has already seen the flag that workgroup 0 sets below
        sum_waves<3, NW>(t, s_dot);
        __syncthreads();
        g = over_waves<NW>(s_dot[0]);
        d = over_waves<NW>(s_dot[1]);
        rr = over_waves<NW>(s_dot[2]);
    }
    if (conv) return;
    const CgStep st = cg_step(i, g, d, rr, gam_old, alpha_old, tol2_bb, bb);
    const double alpha = st.alpha, beta = st.beta;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->gam[i & 1] = g;
        sc->alpha[i & 1] = alpha;
        sc->rr = rr;
        sc->iters = i;
        if (i == 0) sc->rr0 = rr;
        if (st.conv) sc->converged = st.conv;
    }
    if (st.conv || i >= n_max) return;
    if (!kTwin && blockIdx.x == 0)   // read by the previous kernel; the next one adds into it
        for (int k = threadIdx.x; k < 3 * kCgSlots; k += R) cg_buf(cg_slots, i + 2)[k] = 0.0;
    double v[3] = {0.0, 0.0, 0.0};
    auto u_new = [&](double2 w, double s) { return fma(-alpha, fma(beta, s, w.y), w.x); };
    for (;;) {
        const int64_t row = b * R + threadIdx.x;
        const double sj = fma(beta, own_sp.x, own_rw.y);   // D^-1 s
        const double un = fma(-alpha, sj, own_rw.x);       // D^-1 r' = u'
        s_u[threadIdx.x] = un;
#pragma unroll
        for (int k = 0; k < H; ++k)
            if (k * R < bc.stride) s_u[(k + 1) * R + threadIdx.x] = u_new(rw[k], hs[k]);
        for (int k = H * R + threadIdx.x; k < cnt; k += R) {
            const int c = bc.halo[b * bc.stride + k];
            s_u[R + k] = u_new(*reinterpret_cast<const double2*>(V + c), V[c].S);
        }
        __syncthreads();
        double acc;   // (A u')_j
        if (cnt >= 0)
            acc = P.dot(bc, A, [&](unsigned c) { return s_u[c]; });
        else
            acc = P.dot_wide(col, A, [&](int c) { return u_new(*reinterpret_cast<const double2*>(V + c), V[c].S); });
        if (row < n_rows) {
            const double diag = P.a[0];
            const double pj = fma(beta, own_sp.y, own_rw.x);
            x[row] = fma(alpha, pj, own_x);
            double2* o = reinterpret_cast<double2*>(V_new + row);
            o[0] = make_double2(un, acc / diag);
            o[1] = make_double2(sj, pj);
            double dots[3];
            cg_dots(un, acc, diag, dots);
#pragma unroll
            for (int j = 0; j < 3; ++j) v[j] += dots[j];
        }
        if (kTwin) {   // one block per workgroup; s_dot has been read before the barrier above
            sum_waves<3, NW>(v, s_dot);
            __syncthreads();
            if (threadIdx.x < 3) part[(3 * ((i + 1) & 1) + threadIdx.x) * R + b] = over_waves<NW>(s_dot[threadIdx.x]);
            return;
        }
        b += rg.g;
        if (b >= le) break;
        __syncthreads();   // the staged values are read before the next block's
        load();
    }
    block_slot_add<3, R>(v, cg_buf(cg_slots, i + 1));
}

// Values passed between the workgroups of one running kernel: a double as two 64-bit words, a
// float as one, each word with the tag of the iteration it belongs to in the upper half.
// Words are written and read whole, so a reader that sees the tags has the value, whatever
// the order in which stores arrive: no fences, no cache write-backs, no flags.  Written
// through and read past the XCDs' L2s (sc1, device scope), both words in one access; offsets
// in bytes.
struct Mail {
    static constexpr int kDeviceScope = 16;   // sc1
    typedef unsigned v2 __attribute__((ext_vector_type(2)));
    typedef unsigned v4 __attribute__((ext_vector_type(4)));
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Mail(unsigned long long* boxes, unsigned bytes)
        : r(__builtin_amdgcn_make_buffer_rsrc(boxes, 0, (int)bytes, 0x00027000)) {}
    __device__ __forceinline__ void put(unsigned at, double v, unsigned tag) const {
        const v4 w = {(unsigned)__double2loint(v), tag, (unsigned)__double2hiint(v), tag};
        __builtin_amdgcn_raw_buffer_store_b128(w, r, (int)at, 0, kDeviceScope);
    }
    __device__ __forceinline__ void put(unsigned at, float v, unsigned tag) const {
        const v2 w = {__float_as_uint(v), tag};
        __builtin_amdgcn_raw_buffer_store_b64(w, r, (int)at, 0, kDeviceScope);
    }
};

// Copies of the workgroups' partials: every workgroup reads all of one, its XCD's.
constexpr int kSolveCopies = 8;

// K values that a lane waits for.
template <typename S, int K>
struct Inbox {
    static constexpr int kBytes = 2 * sizeof(S);   // of a value in the mail
    unsigned at[K];
    bool need[K];
    unsigned w[K][kBytes / 4];
    __device__ __forceinline__ void expect(int k, unsigned offset, bool n) {
        at[k] = offset;
        need[k] = n;
#pragma unroll
        for (int j = 0; j < kBytes / 4; ++j) w[k][j] = 0;
    }
    __device__ __forceinline__ void load(const Mail& m) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (need[k]) {
                if constexpr (sizeof(S) == 8) {
                    const Mail::v4 v = __builtin_amdgcn_raw_buffer_load_b128(m.r, (int)at[k], 0, Mail::kDeviceScope);
                    w[k][0] = v.x;
                    w[k][1] = v.y;
                    w[k][2] = v.z;
                    w[k][3] = v.w;
                } else {
                    const Mail::v2 v = __builtin_amdgcn_raw_buffer_load_b64(m.r, (int)at[k], 0, Mail::kDeviceScope);
                    w[k][0] = v.x;
                    w[k][1] = v.y;
                }
            }
    }
    __device__ __forceinline__ bool check(unsigned tag) {
        bool ok = true;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (need[k]) {
                if constexpr (sizeof(S) == 8)
                    need[k] = !((w[k][1] == tag) & (w[k][3] == tag));
                else
                    need[k] = w[k][1] != tag;
            }
            ok = ok & !need[k];
        }
        return ok;
    }
    __device__ __forceinline__ S value(int k) const {   // zero where nothing was expected
        if constexpr (sizeof(S) == 8)
            return __hiloint2double((int)w[k][2], (int)w[k][0]);
        else
            return __uint_as_float(w[k][0]);
    }
};

// Polls until every lane of the wave has what it expects of both boxes: a round has all its
// loads in flight together, and a lane sits out for what it has.  Nothing is looked for
// before it can be there, because polls in vain hold up the others' stores.  Waiting 17 x 64
// cycles first (half a microsecond, nearly what a store and a load past the L2s take), 90k
// rows took 3.5 us per Jacobi iteration and 7.9 per FP64 PCG one; without 4.1 and 11.1, with
// 32 x 64 3.7 and 8.5.  Up to 64 workgroups poll so little that 8 are enough (13k rows 2.98
// us, with 16 3.09).  Gives up after `polls` rounds (*fail; at once if there are none).
// Their number comes from LDS, read while the wave sleeps: in a scalar register for the whole
// solve it cost k_pcg_solve<double, 2> 16 more spilled registers and 15% (239k rows).
template <typename A, typename B>
__device__ __forceinline__ void wait_boxes(const Mail& m, A& a, B& b, unsigned tag, int n_wg, const int* s_polls,
                                           int* fail) {
    const int limit = *s_polls;
    if (n_wg > 64)
        __builtin_amdgcn_s_sleep(17);
    else
        __builtin_amdgcn_s_sleep(8);
    const int polls = __builtin_amdgcn_readfirstlane(limit);
    for (int n = 0; n < polls; ++n) {
        asm volatile("" ::: "memory");   // the words are read anew in every round
        a.load(m);
        b.load(m);
        const bool ok = a.check(tag) & b.check(tag);
        if (__all(ok)) return;
    }
    if ((threadIdx.x & 63) == 0) *fail = 1;
}

// A whole Jacobi-PCG solve in one launch, for matrices of which every row block has a
// resident workgroup (launched cooperatively).  The same recurrence and block layout as
// k_cg_iter; the matrix, the block's rows and the halo's (u, s), which the recurrences carry
// along redundantly, stay in registers, so an iteration exchanges one value per row, D^-1 A u,
// and three partial dots per workgroup.  Every workgroup sums all partials in one order (so
// all take the same decisions, and the sums are the same in each run) and that wait is the
// iteration's only grid-wide one.  The boxes are double buffered: a workgroup writes the
// values of iterate i + 2 over those of i after it has seen every partial of i + 1, whose
// writers had read theirs of i.
// Bound by that exchange (a store and a load past the L2s, 0.7 us at least) and the LDS reads
// of the product (0.75 us); what grows with the mesh is the polling, so the partials lie in a
// copy per XCD.  Per iteration against a launch of k_cg_iter: 1.1k rows 5.2 -> 2.7 us, 13k 6.5
// -> 3.0, 90k 7.0 -> 3.5 (registers capped for two workgroups per CU: 0.8 us more, by spills).
// Every wait is bounded: a workgroup that polls `polls` times in vain sets gave_up and
// leaves, those that wait for its next values follow in the same way, and the host solves by
// k_cg_iter<true>, to the same bits.  If it was the last exchange the others finish and report, which is why gave_up
// is a field that only a workgroup giving up writes, and why the iterate goes into an array
// of its own: x, V and the slots are left as they were.
// n_max: the iterate at which the solve stops unconverged.
__global__ __launch_bounds__(kBlockRows) __attribute__((amdgpu_waves_per_eu(2))) void k_cg_solve(
    int64_t n_rows, RowGrid rg, int n_max, const int64_t* __restrict__ sp, BlockCols bc, const double* __restrict__ A,
    const double* __restrict__ x, double* __restrict__ x_out, const CgVec* __restrict__ V, unsigned long long* boxes, unsigned box_bytes, unsigned tag0,
    int polls, const double* __restrict__ cg_slots, CgScalars* sc) {
    extern __shared__ double s_u[];
    constexpr int R = kBlockRows, H = kHaloRegs, NW = R / 64;
    __shared__ double s_dot[3][NW], s_own[3][NW];
    __shared__ int s_fail, s_polls;
    const int64_t b = rg_first(rg);
    if (b >= rg_end(rg)) return;   // the whole workgroup (the grid is a multiple of eight)
    const int nb = (int)bc.nb, tid = threadIdx.x, wave = tid >> 6;
    const int64_t row = b * R + tid, nr = (int64_t)nb * R;
    // boxes: two buffers of a value per row, then two of the workgroups' three partials
    const Mail mail(boxes, box_bytes);
    auto w_box = [&](int buf, int64_t r) { return 16 * (unsigned)(buf * nr + r); };
    auto p_box = [&](int buf, int copy, int k) { return 16 * (unsigned)(2 * nr) + 48 * (unsigned)((buf * kSolveCopies + copy) * nb + k); };
    BlockRow<double> P;
    P.load(bc, b * (R / 64) + wave, sp, A);
    const double tol2_bb = sc->tol2_bb, bb = sc->bb;
    double t[3];
    slot_load_wave<3>(cg_slots, t);
    const int cnt = bc.cnt[b];
    int h[H];
    halo_ids(bc, b, h);
    const int64_t r0 = row < n_rows ? row : 0;
    double u = V[r0].R, w = V[r0].W, s = 0.0, p = 0.0, xr = x[r0];
    double hu[H], hw[H], hs[H];
#pragma unroll
    for (int k = 0; k < H; ++k) {
        hs[k] = hu[k] = hw[k] = 0.0;
        if (k * R < bc.stride) {
            hu[k] = V[h[k]].R;
            hw[k] = V[h[k]].W;
        }
    }
    if (tid == 0) {
        s_fail = 0;
        s_polls = polls;
    }
    double g = wave_total(t[0]), d = wave_total(t[1]), rr = wave_total(t[2]);
    const double rr0 = rr;
    double gam_old = 0.0, alpha_old = 0.0;
    int conv = 0, i = 0;
    for (;; ++i) {
        const CgStep st = cg_step(i, g, d, rr, gam_old, alpha_old, tol2_bb, bb);
        const double alpha = st.alpha, beta = st.beta;
        conv = st.conv;
        if (conv || i >= n_max) break;
        gam_old = g;
        alpha_old = alpha;
        s = __builtin_fma(beta, s, w);             // D^-1 s
        p = __builtin_fma(beta, p, u);
        xr = __builtin_fma(alpha, p, xr);
        u = __builtin_fma(-alpha, s, u);           // D^-1 r'
        s_u[tid] = u;
#pragma unroll
        for (int k = 0; k < H; ++k)
            if (k * R < bc.stride) {
                hs[k] = __builtin_fma(beta, hs[k], hw[k]);
                hu[k] = __builtin_fma(-alpha, hs[k], hu[k]);
                s_u[(k + 1) * R + tid] = hu[k];
            }
        __syncthreads();
        const double acc = P.dot(bc, A, [&](unsigned c) { return s_u[c]; });
        const unsigned tag = tag0 + (unsigned)(i + 1);
        const int buf = (i + 1) & 1;
        double v[3] = {0.0, 0.0, 0.0};
        if (row < n_rows) {
            const double diag = P.a[0];
            w = acc / diag;
            mail.put(w_box(buf, row), w, tag);
            cg_dots(u, acc, diag, v);
        }
        sum_waves<3, NW>(v, s_own);
        __syncthreads();
        if ((tid & 3) < 3 && tid < 4 * kSolveCopies) {
            const int j = tid & 3, copy = tid >> 2;
            mail.put(p_box(buf, copy, (int)b) + 16 * j, over_waves<NW>(s_own[j]), tag);
        }
        // the partials of all workgroups, one per thread, and the halo's values
        Inbox<double, 3> pin;
        Inbox<double, H> win;
#pragma unroll
        for (int j = 0; j < 3; ++j) pin.expect(j, p_box(buf, blockIdx.x % kSolveCopies, min(tid, nb - 1)) + 16 * j, tid < nb);
#pragma unroll
        for (int k = 0; k < H; ++k) win.expect(k, w_box(buf, k * R < bc.stride ? h[k] : 0), k * R + tid < cnt);
        wait_boxes(mail, pin, win, tag, nb, &s_polls, &s_fail);
#pragma unroll
        for (int j = 0; j < 3; ++j) v[j] = pin.value(j);
#pragma unroll
        for (int k = 0; k < H; ++k) hw[k] = win.value(k);
        sum_waves<3, NW>(v, s_dot);
        __syncthreads();
        if (s_fail) {
            if (tid == 0) sc->gave_up = 1;
            return;
        }
        g = over_waves<NW>(s_dot[0]);
        d = over_waves<NW>(s_dot[1]);
        rr = over_waves<NW>(s_dot[2]);
    }
    if (row < n_rows) x_out[row] = xr;
    if (b == 0 && tid == 0) {
        sc->rr = rr;
        sc->rr0 = rr0;
        sc->iters = i;
        sc->converged = conv;
    }
}

// u += the records of one chunk of kNodeSlots incidences, of which every lane of the node's
// quad holds four: the index of the record (padding: the zero record) and, in the top bit,
// whether the node is the edge's tail, which turns the sign of the gradient (component 0)
// and not of the interpolation.
template <typename S>
__device__ __forceinline__ void node_chunk(S u[2], const S* rec, uint2 w, int comp) {
    const unsigned tail = comp == 0 ? 0x8000u : 0u;
    unsigned c[8];
    c[0] = __builtin_amdgcn_mov_dpp((int)w.x, 0x00, 0xf, 0xf, true);   // quad_perm: lane 0 to all four
    c[1] = __builtin_amdgcn_mov_dpp((int)w.y, 0x00, 0xf, 0xf, true);
    c[2] = __builtin_amdgcn_mov_dpp((int)w.x, 0x55, 0xf, 0xf, true);
    c[3] = __builtin_amdgcn_mov_dpp((int)w.y, 0x55, 0xf, 0xf, true);
    c[4] = __builtin_amdgcn_mov_dpp((int)w.x, 0xaa, 0xf, 0xf, true);
    c[5] = __builtin_amdgcn_mov_dpp((int)w.y, 0xaa, 0xf, 0xf, true);
    c[6] = __builtin_amdgcn_mov_dpp((int)w.x, 0xff, 0xf, 0xf, true);
    c[7] = __builtin_amdgcn_mov_dpp((int)w.y, 0xff, 0xf, 0xf, true);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const unsigned lo = c[q] & 0xffffu, hi = c[q] >> 16;
        const S a = rec[4 * (lo & 0x7fffu) + comp], b = rec[4 * (hi & 0x7fffu) + comp];
        u[0] += (lo & tail) ? -a : a;
        u[1] += (hi & tail) ? -b : b;
    }
}

__device__ __forceinline__ uint2 pack(const EdgeVec& t) {
    uint2 w = {0u, 0u};
    __builtin_memcpy(&w, &t, sizeof(EdgeVec));
    return w;
}
__device__ __forceinline__ EdgeVec unpack(uint2 w) {
    EdgeVec t;
    __builtin_memcpy(&t, &w, sizeof(EdgeVec));
    return t;
}

template <typename S>
__device__ __forceinline__ typename Vec<S>::t3 widen(const EdgeVec& t) {
    typename Vec<S>::t3 v;
    v.x = (S)(float)t.x;
    v.y = (S)(float)t.y;
    v.z = (S)(float)t.z;
    return v;
}

// A whole PCG solve with the auxiliary space in one launch: k_cg_solve's scheme for the
// recurrence of k_pcg_q, k_pcg_nodes, k_pcg_fold and k_pcg_update, with kB row blocks and up
// to 2 kB node slices per workgroup.  An iteration has three waits: for q at the slices'
// edges and (p, q); for Y at the row blocks' nodes and the slices' sums of the finest far
// level (further levels are left to the kernels); for z at the halo and (r, z), (r, r).  The
// residual at a slice's edges and p at a block's halo are carried along by the workgroup
// that needs them.  One set of boxes is enough: a value is overwritten in the next iteration
// only after a grid-wide sum whose partials each workgroup gave after it had read the value.
// Bound by the three exchanges (90k rows: 4 of 8 us), then by LDS: the product's reads, the
// slices' sums.  With two blocks the registers hold the matrix and little else; what one
// phase reads is kept in LDS (without that, FP64 spilled 580 bytes per lane: 239k rows 29.9
// us, now 15.5).  Per iteration against the kernels: FP64 1.1k rows 12.0 -> 6.0 us, 51k 13.7
// -> 7.3, 90k 17.8 -> 7.9, 239k 25.0 -> 15.5; FP32 90k 16.3 -> 7.6, beam (246k) 17.6 -> 9.8.
template <typename S, int kB>
__global__ __launch_bounds__(kBlockRows) __attribute__((amdgpu_waves_per_eu(2))) void k_pcg_solve(
    int64_t n_rows, RowGrid rg, int n_max, const int64_t* __restrict__ sp, BlockCols bc, const S* __restrict__ A,
    const S* __restrict__ dinv, const S* x, S* x_out, const typename Vec<S>::t2* __restrict__ ZP,
    const S* __restrict__ R0, AuxSpace g, SolveLists L, unsigned long long* boxes, unsigned box_bytes, unsigned shared_bytes, unsigned tag0,
    int polls, const double* __restrict__ slots, CgScalars* sc) {
    using V4 = typename Vec<S>::t4;
    extern __shared__ __attribute__((aligned(32))) double lds_solve[];
    constexpr int R = kBlockRows, H = kHaloRegs, NW = R / 64, W = 2 * sizeof(S);
    constexpr int E = kSolveEdges / 256, NY = 4 * kSolveNodes / R;   // edges, nodal values per thread
    static_assert(32 * kSolveAggs == R && aux_far_log(0) == 9, "a thread per component and slice of an aggregate");
    __shared__ double s_dot[2][NW], s_own[2][NW], s_far[kB][kSolveAggs][4];
    __shared__ S s_sum[2][4][4];
    __shared__ int s_polls, s_fail, s_fail_y;   // of the waits before a sum over the workgroups, and of the one for Y
    // one after the other in the same memory: p of the blocks and their halos, the slices'
    // records (r', th r') with a zero record, the blocks' nodal values with a zero record
    S* s_p = reinterpret_cast<S*>(lds_solve);
    V4* s_rec = reinterpret_cast<V4*>(lds_solve);
    S* s_y = reinterpret_cast<S*>(lds_solve);
    const int64_t wg = rg_first(rg);
    if (wg >= rg_end(rg)) return;   // the whole workgroup (the grid is a multiple of eight)
    const int nw = (int)rg.nb, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int half = tid >> 8, ht = tid & 255, nl = ht >> 2, comp = tid & 3;
    // the boxes: q and z per row, Y per node and component, the slices' sums, then per copy
    // the workgroups' (p, q), and their (r, z) and (r, r)
    const Mail mail(boxes, box_bytes);
    const unsigned q_box = 0, z_box = W * (unsigned)n_rows, y_box = 2 * z_box, f_box = y_box + 4 * W * (unsigned)g.n_aux,
                   p_box = f_box + 4 * W * (unsigned)L.n_slices;
    auto pq_at = [&](int copy, int k) { return p_box + 16 * (unsigned)(copy * nw + k); };
    auto rz_at = [&](int copy, int k) { return p_box + 16 * (unsigned)(kSolveCopies * nw + 2 * (copy * nw + k)); };
    const int my_copy = blockIdx.x % kSolveCopies;
    const double tol2_bb = sc->tol2_bb, bb = sc->bb;
    double t[2];
    slot_load_wave<2>(slots, t);
    // the row blocks
    // What only one phase of an iteration reads, in LDS behind the rest where a workgroup has
    // several blocks: the edges of its slices with their residuals and vectors, x, D^-1 and
    // (then not in the shared part) p of the rows and the halo.
    constexpr bool kLds = kB > 1;
    const int PS = R + bc.stride, EU = L.stride / 256;
    unsigned char* const s_own_state = reinterpret_cast<unsigned char*>(lds_solve) + shared_bytes;
    uint2* const s_te = reinterpret_cast<uint2*>(s_own_state);
    S* const s_re = reinterpret_cast<S*>(s_te + kB * EU * R);
    S* const s_x = s_re + kB * EU * R;
    S* const s_di = s_x + kB * R;
    if constexpr (kLds) s_p = s_di + kB * R;
    int* const s_e = reinterpret_cast<int*>(s_di + kB * R + kB * PS);
    BlockRow<S> P[kB];
    int row[kB];
    S r[kB], z[kB], hz[kB][H], p1 = S(0), hp1[H], x1 = S(0), di1 = S(0);
    EdgeVec th[kB];
    unsigned en[kB];
    int h[kB][H], cnt[kB], yn[kB][NY], n_node[kB];   // yn: the node, its aggregate's index above bit 24
    S yf[kB][NY];
    const bool far = g.n_far > 0;
    int f_slice[kB];
    const V4* fs = pick<S>(g.far_scale[0], g.far_scale_f[0]);
#pragma unroll
    for (int b = 0; b < kB; ++b) {
        const int64_t blk = wg * kB + b, bl = blk < bc.nb ? blk : bc.nb - 1;
        row[b] = (int)(blk * R + tid);
        P[b].load(bc, blk * NW + wave, sp, A);
        const int rw = row[b] < n_rows ? row[b] : 0;
        r[b] = R0[rw];
        z[b] = ZP[rw].x;
        if constexpr (kLds) {
            s_p[b * PS + tid] = S(0);
            s_x[b * R + tid] = x[rw];
            s_di[b * R + tid] = dinv[rw];
        } else {
            x1 = x[rw];
            di1 = dinv[rw];
        }
        th[b] = g.th[rw];
        en[b] = L.ends[bl * R + tid];
        cnt[b] = blk < bc.nb ? bc.cnt[bl] : 0;
        halo_ids(bc, bl, h[b]);
#pragma unroll
        for (int k = 0; k < H; ++k) {
            hz[b][k] = hp1[k] = S(0);
            if (k * R < bc.stride) {
                hz[b][k] = ZP[h[b][k]].x;
                if constexpr (kLds) s_p[b * PS + (k + 1) * R + tid] = S(0);
            }
        }
        n_node[b] = blk < bc.nb ? L.n_node[bl] : 0;
        const int a0 = L.agg[bl * kSolveAggs + (tid >> 5)];
        f_slice[b] = far && blk < bc.nb && a0 >= 0 ? a0 * 8 + ((tid >> 2) & 7) : L.n_slices;
#pragma unroll
        for (int k = 0; k < NY; ++k) {
            const int64_t at = bl * kSolveNodes + ((tid + k * R) >> 2);
            const int node = L.node[at];
            yn[b][k] = node | (int)L.node_agg[at] << 24;
            yf[b][k] = far ? reinterpret_cast<const S*>(fs + (node >> aux_far_log(0)))[comp] : S(0);
        }
    }
    // the node slices, two at a time (a half of the workgroup each, four lanes per node)
    const int s0 = (int)(wg * L.n_slices / nw), s1 = (int)((wg + 1) * L.n_slices / nw);
    S re1[E], d1[kB], d8[kB], d64[kB];
    EdgeVec te1[E];
    int e1[E], ec[kB];
    uint2 lc[kB];
#pragma unroll
    for (int b = 0; b < kB; ++b) {
        const int sl = s0 + 2 * b + half;
        ec[b] = 0;
        d1[b] = d8[b] = d64[b] = S(0);
        lc[b] = {0u, 0u};
        if constexpr (!kLds) {
#pragma unroll
            for (int k = 0; k < E; ++k) {
                e1[k] = 0;
                re1[k] = S(0);
                te1[k] = EdgeVec{};
            }
        }
        if (sl >= s1) continue;
        ec[b] = L.cnt[sl];
        lc[b] = L.lc[(int64_t)sl * 256 + ht];
#pragma unroll
        for (int k = 0; k < E; ++k)
            if (k * 256 < L.stride) {
                const int ek = L.edge[(int64_t)sl * L.stride + k * 256 + ht];
                if constexpr (kLds) {
                    const int at = (b * EU + k) * R + tid;
                    s_e[at] = ek;
                    s_re[at] = R0[ek];
                    s_te[at] = pack(g.th[ek]);
                } else {
                    e1[k] = ek;
                    re1[k] = R0[ek];
                    te1[k] = g.th[ek];
                }
            }
        const int64_t node = (int64_t)sl * 64 + nl;
        if (node < g.n_aux) {
            d1[b] = reinterpret_cast<const S*>(pick<S>(g.scale, g.scale_f))[4 * node + comp];
            d8[b] = reinterpret_cast<const S*>(pick<S>(g.scale8, g.scale8_f))[4 * (node >> 3) + comp];
            d64[b] = reinterpret_cast<const S*>(pick<S>(g.scale64, g.scale64_f))[4 * (int64_t)sl + comp];
        }
    }
    if (tid == 0) {
        s_fail = s_fail_y = 0;
        s_polls = polls;
    }
    double gm = wave_total(t[0]), rr = wave_total(t[1]);
    const double rr0 = rr;
    double gam_old = 0.0;
    int conv = 0, i = 0;
    // the workgroup's sums of n values into every copy of its partials
    auto give = [&](const double* v, int n, unsigned tag) {
        for (int j = 0; j < n; ++j) {
            const double a = wave_total(v[j]);
            if (lane == 0) s_own[j][wave] = a;
        }
        __syncthreads();
        const int j = tid & 1, copy = tid >> 1;
        if (j < n && copy < kSolveCopies) {
            double a = 0.0;
#pragma unroll
            for (int q = 0; q < NW; ++q) a += s_own[j][q];
            mail.put(n == 1 ? pq_at(copy, (int)wg) : rz_at(copy, (int)wg) + 16 * j, a, tag);
        }
    };
    // all workgroups' partials, one per thread, summed in one order; false: given up
    auto sum = [&](double* v, int n) {
        for (int j = 0; j < n; ++j) {
            const double a = wave_total(v[j]);
            if (lane == 0) s_dot[j][wave] = a;
        }
        __syncthreads();
        for (int j = 0; j < n; ++j) {
            v[j] = 0.0;
#pragma unroll
            for (int q = 0; q < NW; ++q) v[j] += s_dot[j][q];
        }
        return s_fail == 0;
    };
    for (;; ++i) {
        const bool done = !(rr > tol2_bb) || bb == 0.0;
        const double beta = (i == 0) ? 0.0 : gm / gam_old;
        const bool bad = !done && !(gm > 0.0 && gm < INFINITY && beta >= 0.0 && beta < INFINITY);
        conv = done ? 1 : (bad ? 2 : 0);
        if (conv || i >= n_max) break;
        gam_old = gm;
        const unsigned tag = tag0 + (unsigned)(i + 1);
        const S bs = (S)beta;
        // q = A p
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            S* sb = s_p + b * PS + tid;
            if constexpr (kLds) {
                sb[0] = fma(bs, sb[0], z[b]);
#pragma unroll
                for (int k = 0; k < H; ++k)
                    if (k * R < bc.stride) sb[(k + 1) * R] = fma(bs, sb[(k + 1) * R], hz[b][k]);
            } else {
                sb[0] = p1 = fma(bs, p1, z[b]);
#pragma unroll
                for (int k = 0; k < H; ++k)
                    if (k * R < bc.stride) sb[(k + 1) * R] = hp1[k] = fma(bs, hp1[k], hz[b][k]);
            }
        }
        __syncthreads();
        S q[kB];
        double v[2] = {0.0, 0.0};
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            const S* sb = s_p + b * PS;
            q[b] = P[b].dot(bc, A, [&](unsigned c) { return sb[c]; });
            if (row[b] < n_rows) {
                mail.put(q_box + W * (unsigned)row[b], q[b], tag);
                v[0] += (double)(kLds ? sb[tid] : p1) * (double)q[b];
            }
        }
        give(v, 1, tag);
        {
            Inbox<double, 1> pin;
            pin.expect(0, pq_at(my_copy, min(tid, nw - 1)), tid < nw);
            Inbox<S, kB * E> qin;
#pragma unroll
            for (int k = 0; k < kB * E; ++k) {
                const bool need = (k % E) * 256 + ht < ec[k / E];
                int ek = 0;
                if constexpr (kLds) {
                    if (need) ek = s_e[(k / E * EU + k % E) * R + tid];
                } else {
                    ek = e1[k % E];
                }
                qin.expect(k, q_box + W * (unsigned)ek, need);
            }
            wait_boxes(mail, pin, qin, tag, nw, &s_polls, &s_fail);
            v[0] = pin.value(0);
            if (!sum(v, 1)) break;
            const double alpha = gm / v[0];
            if (!(alpha > 0.0 && alpha < INFINITY)) {
                conv = 2;
                break;
            }
            const S as = (S)alpha;
#pragma unroll
            for (int b = 0; b < kB; ++b) {
                if constexpr (kLds)
                    s_x[b * R + tid] = fma(as, s_p[b * PS + tid], s_x[b * R + tid]);
                else
                    x1 = fma(as, p1, x1);
                r[b] = fma(-as, q[b], r[b]);
            }
#pragma unroll
            for (int k = 0; k < kB * E; ++k) {
                if constexpr (kLds) {
                    if ((k % E) * 256 + ht < ec[k / E]) {
                        S& re = s_re[(k / E * EU + k % E) * R + tid];
                        re = fma(-as, qin.value(k), re);
                    }
                } else {
                    re1[k % E] = fma(-as, qin.value(k), re1[k % E]);
                }
            }
        }
        // the slices' nodal sums
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            if (s0 + 2 * b >= s1) break;   // the whole workgroup
            const int sl = s0 + 2 * b + half;
            const bool mine = sl < s1;     // the whole wave
            V4* rec4 = s_rec + half * (L.stride + 1);
            if (mine) {
#pragma unroll
                for (int k = 0; k < E; ++k)
                    if (k * 256 < L.stride) {
                        S rk;
                        EdgeVec tk;
                        if constexpr (kLds) {
                            const int at = (b * EU + k) * R + tid;
                            rk = s_re[at];
                            tk = unpack(s_te[at]);
                        } else {
                            rk = re1[k];
                            tk = te1[k];
                        }
                        const auto tv = widen<S>(tk);
                        rec4[k * 256 + ht] = Vec<S>::four(rk, tv.x * rk, tv.y * rk, tv.z * rk);
                    }
                if (ht == 0) rec4[L.stride] = Vec<S>::four(S(0), S(0), S(0), S(0));
            }
            __syncthreads();
            S own = S(0), s8 = S(0);
            if (mine) {
                const S* rec = reinterpret_cast<const S*>(rec4);
                S u[2] = {S(0), S(0)};
                node_chunk<S>(u, rec, lc[b], comp);
                for (int k = L.n_extra ? L.xsp[sl] : 0, k1 = L.n_extra ? L.xsp[sl + 1] : 0; k < k1; ++k)
                    node_chunk<S>(u, rec, L.xlc[(int64_t)k * 256 + ht], comp);
                own = s8 = u[0] + u[1];   // zero for the padding nodes of the last slice
                s8 += __shfl_xor(s8, 4);
                s8 += __shfl_xor(s8, 8);
                s8 += __shfl_xor(s8, 16);
                const S s16 = s8 + __shfl_xor(s8, 32);
                if (lane < 4) s_sum[half][wave & 3][lane] = s16;
            }
            __syncthreads();
            if (mine) {
                S s64 = S(0);
#pragma unroll
                for (int k = 0; k < 4; ++k) s64 += s_sum[half][k][comp];
                const int64_t node = (int64_t)sl * 64 + nl;
                const S y = own * d1[b] + s8 * d8[b] + s64 * d64[b];
                if (node < g.n_aux) mail.put(y_box + W * (4 * (unsigned)node + comp), y, tag);
                if (far && ht < 4) mail.put(f_box + W * (4 * (unsigned)sl + comp), s64, tag);
            }
        }
        // Y with the far level at the blocks' nodes
        {
            Inbox<S, kB * NY> yin;
            Inbox<S, kB> fin;
#pragma unroll
            for (int k = 0; k < kB * NY; ++k)
                yin.expect(k, y_box + W * (4 * ((unsigned)yn[k / NY][k % NY] & 0xffffffu) + comp),
                           ((tid + (k % NY) * R) >> 2) < n_node[k / NY]);
#pragma unroll
            for (int b = 0; b < kB; ++b) {
                const bool need = f_slice[b] < L.n_slices;
                fin.expect(b, f_box + W * (4 * (unsigned)(need ? f_slice[b] : 0) + comp), need);
            }
            wait_boxes(mail, yin, fin, tag, nw, &s_polls, &s_fail_y);
            if (far) {
#pragma unroll
                for (int b = 0; b < kB; ++b) {
                    double f = (double)fin.value(b);   // the aggregate's eight slices
                    f += __shfl_xor(f, 4);
                    f += __shfl_xor(f, 8);
                    f += __shfl_xor(f, 16);
                    if ((tid & 28) == 0) s_far[b][tid >> 5][comp] = f;
                }
                __syncthreads();
            }
#pragma unroll
            for (int k = 0; k < kB * NY; ++k) {
                const int b = k / NY, kk = k % NY;
                S y = yin.value(k);
                if (far) y += (S)s_far[b][(unsigned)yn[b][kk] >> 24][comp] * yf[b][kk];
                s_y[b * 4 * (kSolveNodes + 1) + tid + kk * R] = y;
            }
            if (tid < 4 * kB) s_y[(tid >> 2) * 4 * (kSolveNodes + 1) + 4 * kSolveNodes + comp] = S(0);
            __syncthreads();
            if (s_fail_y) break;
        }
        // z and its dots
        v[0] = v[1] = 0.0;
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            const V4* yb = reinterpret_cast<const V4*>(s_y) + b * (kSolveNodes + 1);
            const V4 y0 = yb[en[b] & 0xffffu], y1 = yb[en[b] >> 16];
            const auto tv = widen<S>(th[b]);
            S di;
            if constexpr (kLds)
                di = s_di[b * R + tid];
            else
                di = di1;
            z[b] = di * r[b] + (y1.x - y0.x) + tv.x * (y0.y + y1.y) + tv.y * (y0.z + y1.z) + tv.z * (y0.w + y1.w);
            if (row[b] < n_rows) {
                mail.put(z_box + W * (unsigned)row[b], z[b], tag);
                v[0] += (double)r[b] * (double)z[b];
                v[1] += (double)r[b] * (double)r[b];
            }
        }
        give(v, 2, tag);
        {
            Inbox<double, 2> pin;
            pin.expect(0, rz_at(my_copy, min(tid, nw - 1)), tid < nw);
            pin.expect(1, rz_at(my_copy, min(tid, nw - 1)) + 16, tid < nw);
            Inbox<S, kB * H> zin;
#pragma unroll
            for (int k = 0; k < kB * H; ++k)
                zin.expect(k, z_box + W * (unsigned)((k % H) * R < bc.stride ? h[k / H][k % H] : 0),
                           (k % H) * R + tid < cnt[k / H]);
            wait_boxes(mail, pin, zin, tag, nw, &s_polls, &s_fail);
            v[0] = pin.value(0);
            v[1] = pin.value(1);
            if (!sum(v, 2)) break;
            gm = v[0];
            rr = v[1];
#pragma unroll
            for (int k = 0; k < kB * H; ++k) hz[k / H][k % H] = zin.value(k);
        }
    }
    if (s_fail || s_fail_y) {   // the same for the whole workgroup: a barrier follows every wait
        if (tid == 0) sc->gave_up = 1;
        return;
    }
#pragma unroll
    for (int b = 0; b < kB; ++b)
        if (row[b] < n_rows) x_out[row[b]] = kLds ? s_x[b * R + tid] : x1;
    if (wg == 0 && tid == 0) {
        sc->rr = rr;
        sc->rr0 = rr0;
        sc->iters = i;
        sc->converged = conv;
    }
}

// ||b||^2 from the partials of the kernel that summed it (the right-hand side's, or the
// true residual's for an inner solve); r = b - A x, or with zero_x r = b and x = 0 (the
// inner solves start from zero); q = 0; clears the four reduction buffers and the far
// levels' accumulators.
template <typename S>
__global__ __launch_bounds__(kBlock) void k_pcg_init(int64_t n_rows, RowGrid rg, const int64_t* __restrict__ sp,
                                                      const int32_t* __restrict__ col, const S* __restrict__ A,
                                                      const double* __restrict__ b, S* __restrict__ x, bool zero_x,
                                                      S* __restrict__ R, S* __restrict__ Q,
                                                      const double* __restrict__ part_b, double* cg_slots,
                                                      CgScalars* sc, double tol, AuxSpace g) {
    double bb[1];
    read_partials<1>(part_b, gridDim.x, bb);
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            sc->bb = bb[0];
            sc->tol2_bb = tol * tol * bb[0];
            sc->converged = 0;
            sc->gave_up = 0;
        }
        for (int k = threadIdx.x; k < 4 * 3 * kCgSlots; k += kBlock) cg_slots[k] = 0.0;
        clear_far(g);
    }
    for (int64_t lb = rg_first(rg), le = rg_end(rg); lb < le; lb += rg.g) {
        const int64_t row = lb * kBlock + threadIdx.x;
        if (((row >> 6) << 6) >= n_rows) continue;
        if (zero_x) {
            if (row < n_rows) {
                R[row] = (S)b[row];
                Q[row] = S(0);
                x[row] = S(0);
            }
            continue;
        }
        if constexpr (sizeof(S) == 8) {
            const double ax = sell_row(sp, col, A, row, [&](int c) { return x[c]; });
            if (row < n_rows) {
                R[row] = b[row] - ax;
                Q[row] = 0.0;
            }
        }
    }
}

// The convergence test of iterate i (its (r, r) from reduction 2i - 1), beta, the new
// direction p = z + beta p and q = A p (only q is stored: the update kernel forms the same
// p from the same operands); (p, q) into reduction 2i.
// One workgroup per row block.  Bound by HBM on the large meshes, by the chain of dependent
// loads on the small ones; both were set by the gathers (per stored slot a 32-bit column,
// then a (z, p) pair from L2, six slots at a time: up to twelve round trips in a row).
// Staging p of the block's own and halo columns in LDS leaves one round trip (list, pairs)
// beside the matrix stream, 6 instead of 8 bytes per FP32 slot, and one LDS read per slot.
// FP32: 998k tets 31.2 -> 23.6 us (about 150 MB: 6.4 TB/s), 384k tets 16.6 -> 12.4, beam
// 11.8 -> 7.9; FP64: 197k tets 13.8 -> 10.8, 73k 7.7 -> 6.1, 41k 6.4 -> 5.8.
template <typename S>
__global__ __launch_bounds__(kBlockRows) void k_pcg_q(int64_t n_rows, RowGrid rg, int i, const int64_t* __restrict__ sp,
                                             const int32_t* __restrict__ col, BlockCols bc, const S* __restrict__ A,
                                             const typename Vec<S>::t2* __restrict__ ZP, S* __restrict__ Q,
                                             double* __restrict__ cg_slots, CgScalars* sc, AuxSpace aux) {
    using V2 = typename Vec<S>::t2;
    extern __shared__ double lds_raw[];
    S* s_p = reinterpret_cast<S*>(lds_raw);
    constexpr int R = kBlockRows, H = kHaloRegs;
    const int conv = sc->converged;
    const double tol2_bb = sc->tol2_bb, bb = sc->bb, gam_old = sc->gam[(i + 1) & 1];
    double t[2];
    slot_load_wave<2>(red_buf(cg_slots, 2 * i - 1), t);
    const int64_t b = rg_first(rg);
    if (b >= rg_end(rg)) return;   // the whole workgroup
    const int64_t row = b * R + threadIdx.x;
    // in flight together: the row's values and indices, its own pair, and the halo's
    BlockRow<S> P;
    P.load(bc, b * (R / 64) + (threadIdx.x >> 6), sp, A);
    const V2 own = ZP[row < n_rows ? row : 0];
    const int cnt = bc.cnt[b];
    int h[H];
    halo_ids(bc, b, h);
    V2 zp[H];
#pragma unroll
    for (int k = 0; k < H; ++k)
        if (k * R < bc.stride) zp[k] = ZP[h[k]];
    if (conv) return;
    const double g = wave_total(t[0]), rr = wave_total(t[1]);
    const bool done = !(rr > tol2_bb) || bb == 0.0;
    const double beta = (i == 0) ? 0.0 : g / gam_old;
    const bool bad = !done && !(g > 0.0 && g < INFINITY && beta >= 0.0 && beta < INFINITY);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->gam[i & 1] = g;
        sc->rr = rr;
        sc->iters = i;
        if (i == 0) sc->rr0 = rr;
        if (done) sc->converged = 1;
        if (bad) sc->converged = 2;
    }
    if (done || bad) return;
    if (blockIdx.x == 0) clear_far(aux);   // read by the previous update, added to by the next node pass
    const S bs = (S)beta;
    const S p = own.x + bs * own.y;
    s_p[threadIdx.x] = p;
#pragma unroll
    for (int k = 0; k < H; ++k)
        if (k * R < bc.stride) s_p[(k + 1) * R + threadIdx.x] = zp[k].x + bs * zp[k].y;
    for (int k = H * R + threadIdx.x; k < cnt; k += R) {
        const V2 v = ZP[bc.halo[b * bc.stride + k]];
        s_p[R + k] = v.x + bs * v.y;
    }
    __syncthreads();
    S q;
    if (cnt >= 0) {
        q = P.dot(bc, A, [&](unsigned c) { return s_p[c]; });
    } else {
        q = P.dot_wide(col, A, [&](int c) {
            const V2 v = ZP[c];
            return v.x + bs * v.y;
        });
    }
    double v[1] = {0.0};
    if (row < n_rows) {
        Q[row] = q;
        v[0] = (double)p * (double)q;
    }
    block_slot_add<1, R>(v, red_buf(cg_slots, 2 * i));
}

// Sums over a node's edges of s_e r_e, s_e q_e, th_e r_e and th_e q_e (r' = r - alpha q is
// formed once alpha is known).  A workgroup takes one slice of 64 nodes: wave j sums
// slots j, j + 4, j + 8, ... of every node (coalesced loads of the slice's columns), and
// the four partial sums meet in LDS.  Padding entries read edge 0 and count zero.
constexpr int kNodePhases = kBlock / 64;

template <typename S>
__device__ __forceinline__ void node_part(S P[8], const AuxSpace& g, const S* __restrict__ R,
                                          const S* __restrict__ Q, int64_t sl, int lane, int j) {
    const int64_t k0 = g.sp[sl] + lane, k1 = g.sp[sl + 1];
#pragma unroll
    for (int v = 0; v < 8; ++v) P[v] = S(0);
    constexpr int U = 4;   // slots per thread in flight together (about all of a node's share)
    for (int64_t k = k0 + 64 * j; k < k1; k += U * kNodePhases * 64) {
        int32_t c[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int64_t kk = k + (int64_t)q * kNodePhases * 64;
            c[q] = kk < k1 ? g.inc[kk] : kAuxPad;
        }
        S rv[U], qv[U];
        typename Vec<S>::t3 th[U];
        S s[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const bool ok = c[q] != kAuxPad;
            const int32_t e = ok ? (c[q] >= 0 ? c[q] : ~c[q]) : 0;
            s[q] = ok ? (c[q] >= 0 ? S(1) : S(-1)) : S(0);
            rv[q] = R[e];
            qv[q] = Q[e];
            th[q] = edge_vec_t<S>(g, e);
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const S r = s[q] != S(0) ? rv[q] : S(0), qq = s[q] != S(0) ? qv[q] : S(0);
            P[0] += s[q] * r;
            P[1] += s[q] * qq;
            P[2] += th[q].x * r;
            P[3] += th[q].y * r;
            P[4] += th[q].z * r;
            P[5] += th[q].x * qq;
            P[6] += th[q].y * qq;
            P[7] += th[q].z * qq;
        }
    }
}

// alpha from reduction 2i (i = -1: the start, alpha = 0); Y = (D_G^-1 G^T r', D_Pi^-1 Pi^T r').
// rg runs over slices of 64 nodes.
template <typename S>
__global__ __launch_bounds__(kBlock) void k_pcg_nodes(RowGrid rg, int i, AuxSpace g, const S* __restrict__ R,
                                                       const S* __restrict__ Q, double* __restrict__ cg_slots,
                                                       CgScalars* sc) {
    __shared__ S part[8][kNodePhases][64];
    const int conv = sc->converged;
    const double gam = sc->gam[i & 1];
    double t[1] = {0.0};
    if (i >= 0) slot_load_wave<1>(red_buf(cg_slots, 2 * i), t);
    const int lane = threadIdx.x & 63, j = threadIdx.x >> 6;
    const int nl = threadIdx.x >> 2, comp = threadIdx.x & 3;   // output: node of the slice, component
    int64_t sl = rg_first(rg);
    const int64_t le = rg_end(rg);
    const S* scale = reinterpret_cast<const S*>(pick<S>(g.scale, g.scale_f));
    const S* scale8 = reinterpret_cast<const S*>(pick<S>(g.scale8, g.scale8_f));
    const S* scale64 = reinterpret_cast<const S*>(pick<S>(g.scale64, g.scale64_f));
    // the output's three scales, loaded with the slice's incidences (they depend on nothing
    // else, and would otherwise be a memory round trip of their own after the barrier)
    S d1 = S(0), d8 = S(0), d64 = S(0);
    auto load_scales = [&](int64_t s) {
        const int64_t node = s * 64 + nl;
        if (node < g.n_aux) {
            d1 = scale[4 * node + comp];
            d8 = scale8[4 * (node >> 3) + comp];
            d64 = scale64[4 * s + comp];
        }
    };
    S P[8];
    if (sl < le) {
        load_scales(sl);
        node_part<S>(P, g, R, Q, sl, lane, j);
    }
    if (conv) return;
    double alpha = 0.0;
    if (i >= 0) {
        alpha = gam / wave_total(t[0]);
        if (!(alpha > 0.0 && alpha < INFINITY)) {
            if (blockIdx.x == 0 && threadIdx.x == 0) sc->converged = 2;
            return;
        }
    }
    if (blockIdx.x == 0) clear_buf(red_buf(cg_slots, 2 * i + 1));
    const S as = (S)alpha;
    S* Y = reinterpret_cast<S*>(pick<S>(g.Y, g.Y_f));
    __shared__ S wsum[kNodePhases][4];
    // component comp of P^T r' at node nl: (sum of value va) - alpha (sum of value vb)
    const int va = comp == 0 ? 0 : 1 + comp, vb = comp == 0 ? 1 : 4 + comp;
    while (sl < le) {
#pragma unroll
        for (int v = 0; v < 8; ++v) part[v][j][lane] = P[v];
        __syncthreads();
        const int64_t node = sl * 64 + nl;
        S a = S(0), b = S(0);
#pragma unroll
        for (int q = 0; q < kNodePhases; ++q) {
            a += part[va][q][nl];
            b += part[vb][q][nl];
        }
        const S u = a - as * b;   // zero for the padding nodes of the last slice
        // the aggregate of 8 nodes: lanes 4 nl + comp with the same comp and nl >> 3
        S s8 = u;
        s8 += __shfl_xor(s8, 4);
        s8 += __shfl_xor(s8, 8);
        s8 += __shfl_xor(s8, 16);
        // the aggregate of 64 nodes (the slice): the wave's two groups, then the four waves
        S s16 = s8 + __shfl_xor(s8, 32);
        if (lane < 4) wsum[j][lane] = s16;
        __syncthreads();
        S s64 = S(0);
#pragma unroll
        for (int q = 0; q < kNodePhases; ++q) s64 += wsum[q][comp];
        if (node < g.n_aux) Y[4 * node + comp] = u * d1 + s8 * d8 + s64 * d64;
        // Far levels: the slice's sums added into its aggregate of the finest far level
        // (each component of an aggregate has its own 64-byte line, so eight workgroups add
        // into one line); the coarser far levels' sums are formed from those by the fold.
        if (threadIdx.x < 4 && g.n_far > 0)   // comp = threadIdx.x
            unsafeAtomicAdd(far_line(g, (sl * 64) >> aux_far_log(0), comp), (double)s64);
        __syncthreads();
        sl += rg.g;
        if (sl < le) {
            load_scales(sl);
            node_part<S>(P, g, R, Q, sl, lane, j);
        }
    }
}

// A row's own values for the update.
template <typename S>
struct UPart {
    S r, q;
    typename Vec<S>::t2 zp;
    S x, dinv;
    typename Vec<S>::t3 th;
    typename Vec<S>::t4 ya, yb;
};

template <typename S>
__device__ __forceinline__ void u_part(UPart<S>& P, const AuxSpace& g, const S* __restrict__ dinv,
                                       const S* __restrict__ x, const typename Vec<S>::t2* __restrict__ ZP,
                                       const S* __restrict__ R, const S* __restrict__ Q, int64_t row) {
    P.r = R[row];
    P.q = Q[row];
    P.zp = ZP[row];
    P.x = x[row];
    P.dinv = dinv[row];
    P.th = edge_vec_t<S>(g, row);
    const int2 en = g.ends[row];
    const typename Vec<S>::t4* Y = pick<S>(g.Y, g.Y_f);
    P.ya = Y[en.x];   // the far levels' corrections are already folded in (k_pcg_fold)
    P.yb = Y[en.y];
}

// The far levels' corrections folded into each node's Y once, after the node pass has
// summed the finest far level's aggregates and before the update reads Y at both ends of
// every edge: Y += (the aggregate's sum) * (its scale), level by level.  The coarser
// levels' sums are those of their eight (level 1) and 64 (level 2) finest aggregates: a
// workgroup's 256 nodes lie in one aggregate of each far level, so thread t loads
// component t & 3 of the (t >> 2)-th finest aggregate of its level-2 aggregate, groups of
// eight are summed across lanes and the groups in LDS.
template <typename S>
__global__ __launch_bounds__(kBlock) void k_pcg_fold(AuxSpace g, const CgScalars* __restrict__ sc) {
    static_assert(kBlock == 256 && aux_far_log(0) >= 8 && aux_far_log(1) == aux_far_log(0) + 3 &&
                      aux_far_log(2) == aux_far_log(0) + 6 && kAuxFarLevels == 3,
                  "one workgroup's nodes in one aggregate per far level; 8 and 64 finest ones per coarser");
    if (sc->converged) return;   // a stopped solve's node pass left Y as it was (uniform)
    const int64_t n0 = (int64_t)blockIdx.x * kBlock, n = n0 + threadIdx.x;
    double c1[4] = {0.0, 0.0, 0.0, 0.0}, c2[4] = {0.0, 0.0, 0.0, 0.0};
    if (g.n_far > 1) {
        __shared__ double grp[8][4];
        const int comp = threadIdx.x & 3, lane = threadIdx.x & 63;
        const int64_t nf0 = (g.n_aux + (1ll << aux_far_log(0)) - 1) >> aux_far_log(0);
        const int64_t a = ((n0 >> aux_far_log(2)) << 6) + (threadIdx.x >> 2);
        double v = a < nf0 ? *far_line(g, a, comp) : 0.0;
        v += __shfl_xor(v, 4);    // lanes 4k + comp: the eight consecutive k of one group
        v += __shfl_xor(v, 8);
        v += __shfl_xor(v, 16);
        if ((lane & 28) == 0) grp[threadIdx.x >> 5][comp] = v;   // group (threadIdx.x >> 2) >> 3
        __syncthreads();
        const int q1 = (int)((n0 >> aux_far_log(1)) & 7);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            c1[c] = grp[q1][c];
            double t = 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) t += grp[q][c];
            c2[c] = t;
        }
    }
    if (n >= g.n_aux) return;
    typename Vec<S>::t4* Y = pick<S>(g.Y, g.Y_f);
    typename Vec<S>::t4 y = Y[n];
#pragma unroll
    for (int L = 0; L < kAuxFarLevels; ++L) {
        if (L >= g.n_far) break;
        const typename Vec<S>::t4* fs = pick<S>(g.far_scale[L], g.far_scale_f[L]);
        const int64_t a = n >> aux_far_log(L);
        const typename Vec<S>::t4 d = fs[a];
        double f[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) f[c] = L == 0 ? *far_line(g, a, c) : (L == 1 ? c1[c] : c2[c]);
        y.x += (S)f[0] * d.x;
        y.y += (S)f[1] * d.y;
        y.z += (S)f[2] * d.z;
        y.w += (S)f[3] * d.w;
    }
    Y[n] = y;
}

// x += alpha p with p = z + beta p from the pair k_pcg_q(i) read (not at the start),
// r' = r - alpha q, z' = D^-1 r' + G y + Pi v; the pair (z', p) into the other buffer;
// (r', z') and (r', r') into reduction 2i + 1.  Each workgroup takes one block of kR
// consecutive groups of kBlock rows (the grid covers all rows), and each thread issues the
// loads of its kR rows together: the FP32 form, whose rows carry fewer bytes, takes two.
template <typename S, int kR>
__global__ __launch_bounds__(kBlock) void k_pcg_update(int64_t n_rows, RowGrid rg, int i, AuxSpace g,
                                                        const S* __restrict__ dinv, S* __restrict__ x,
                                                        const typename Vec<S>::t2* __restrict__ ZP,
                                                        typename Vec<S>::t2* __restrict__ ZPn, S* __restrict__ R,
                                                        const S* __restrict__ Q, double* __restrict__ cg_slots,
                                                        CgScalars* sc) {
    const int conv = sc->converged;
    const double gam = sc->gam[i & 1], gam_old = sc->gam[(i + 1) & 1];
    double t[1] = {0.0};
    if (i >= 0) slot_load_wave<1>(red_buf(cg_slots, 2 * i), t);
    const int64_t lb = rg_first(rg);
    const int64_t le = rg_end(rg);
    UPart<S> P[kR];
    bool act[kR];
#pragma unroll
    for (int k = 0; k < kR; ++k) {
        const int64_t row = (lb * kR + k) * kBlock + threadIdx.x;
        act[k] = lb < le && row < n_rows;
        if (act[k]) u_part<S>(P[k], g, dinv, x, ZP, R, Q, row);
    }
    if (conv) return;
    double alpha = 0.0;
    if (i >= 0) {
        alpha = gam / wave_total(t[0]);
        if (!(alpha > 0.0 && alpha < INFINITY)) return;
    }
    // beta of this iteration, from the same operands as in k_pcg_q (the same bits)
    const double beta = (i <= 0) ? 0.0 : gam / gam_old;
    if (blockIdx.x == 0) clear_buf(red_buf(cg_slots, 2 * i + 2));
    const S as = (S)alpha, bs = (S)beta;
    double v[2] = {0.0, 0.0};
#pragma unroll
    for (int k = 0; k < kR; ++k) {
        if (!act[k]) continue;
        const int64_t row = (lb * kR + k) * kBlock + threadIdx.x;
        const UPart<S>& U = P[k];
        const S r = U.r - as * U.q;
        const S p = i >= 0 ? U.zp.x + bs * U.zp.y : S(0);
        if (i >= 0) x[row] = U.x + as * p;
        const S z = U.dinv * r + (U.yb.x - U.ya.x) + U.th.x * (U.ya.y + U.yb.y) + U.th.y * (U.ya.z + U.yb.z) +
                    U.th.z * (U.ya.w + U.yb.w);
        R[row] = r;
        ZPn[row] = Vec<S>::two(z, p);
        v[0] += (double)r * (double)z;
        v[1] += (double)r * (double)r;
    }
    block_slot_add<2, kBlock>(v, red_buf(cg_slots, 2 * i + 1));
}

// Rows per thread of the update kernel.
template <typename S>
constexpr int update_rows() { return sizeof(S) == 4 ? 2 : 1; }

// ||b||^2 and the tolerance from the right-hand side's partials (one workgroup).
__global__ __launch_bounds__(kBlock) void k_rhs_norm(const double* __restrict__ part_b, int n_src, CgScalars* sc,
                                                      double tol) {
    double bb[1];
    read_partials<1>(part_b, n_src, bb);
    if (threadIdx.x == 0) {
        sc->bb = bb[0];
        sc->tol2_bb = tol * tol * bb[0];
        sc->converged = 0;
    }
}

// FP32 copy of n values; x += d (FP64 from FP32).
__global__ __launch_bounds__(kBlock) void k_to_f32(const double* __restrict__ a, float* __restrict__ b, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) b[i] = (float)a[i];
}

__global__ __launch_bounds__(kBlock) void k_add_f32(double* __restrict__ x, const float* __restrict__ d, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) x[i] += (double)d[i];
}

__global__ __launch_bounds__(kBlock) void k_zero_if_b_zero(double* x, int64_t n, const CgScalars* sc) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n && sc->bb == 0.0) x[i] = 0.0;
}

__global__ __launch_bounds__(kBlock) void k_cg_resid(int64_t n_rows, RowGrid rg, const int64_t* __restrict__ sp,
                                                      const int32_t* __restrict__ col, const double* __restrict__ A,
                                                      const double* __restrict__ b, const double* __restrict__ x,
                                                      double* __restrict__ rt, double* __restrict__ partial) {
    double v[1] = {0.0};
    for (int64_t lb = rg_first(rg), le = rg_end(rg); lb < le; lb += rg.g) {
        const int64_t row = lb * kBlock + threadIdx.x;
        if (((row >> 6) << 6) >= n_rows) continue;
        const double ax = sell_row(sp, col, A, row, [&](int c) { return x[c]; });
        if (row < n_rows) {
            const double d = b[row] - ax;
            rt[row] = d;
            v[0] += d * d;
        }
    }
    write_partials<1>(v, partial);
}

// One workgroup: sum n_src partials into *out.
__global__ __launch_bounds__(kBlock) void k_finalize(const double* __restrict__ partial, int n_src, double* out) {
    double t[1];
    read_partials<1>(partial, n_src, t);
    if (threadIdx.x == 0) *out = t[0];
}

// b_new = b_old - dt C (gamma e_new + (1 - gamma) e_old); face (i,j,k) has edges
// (i,j) +1, (j,k) +1, (i,k) -1.
__global__ __launch_bounds__(kBlock) void k_faraday(int64_t n_faces, const int32_t* __restrict__ fe,
                                                     const double* __restrict__ b_old,
                                                     const double* __restrict__ e_new,
                                                     const double* __restrict__ e_old, double dt, double gamma,
                                                     double* __restrict__ b_new) {
    int64_t f = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (f >= n_faces) return;
    const int a = fe[3 * f], b = fe[3 * f + 1], c = fe[3 * f + 2];
    const double ea = gamma * e_new[a] + (1.0 - gamma) * e_old[a];
    const double eb = gamma * e_new[b] + (1.0 - gamma) * e_old[b];
    const double ec = gamma * e_new[c] + (1.0 - gamma) * e_old[c];
    b_new[f] = b_old[f] - dt * (ea + eb - ec);
}

// out[node] += D^T v: +v at the head, -v at the tail of every edge.
__global__ __launch_bounds__(kBlock) void k_DT(int64_t n_edges, const int32_t* __restrict__ edges,
                                                const double* __restrict__ v, double* __restrict__ out) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n_edges) return;
    const double x = v[i];
    if (x != 0.0) {
        unsafeAtomicAdd(out + edges[2 * i + 1], x);
        unsafeAtomicAdd(out + edges[2 * i], -x);
    }
}

// Largest |v| over the workgroup (values as ordered bit patterns), then one atomicMax by
// thread 0: same-address atomics from every thread would serialize at the memory side.
template <int NV>
__device__ __forceinline__ void block_max_abs(const double v[NV], unsigned long long* const out[NV]) {
    __shared__ unsigned long long s[NV][kBlock / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        unsigned long long m = (unsigned long long)__double_as_longlong(fabs(v[j]));
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const unsigned long long o = __shfl_xor(m, off);
            m = o > m ? o : m;
        }
        if (lane == 0) s[j][w] = m;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            unsigned long long m = 0;
            for (int q = 0; q < kBlock / 64; ++q) m = s[j][q] > m ? s[j][q] : m;
            if (m) atomicMax(out[j], m);
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_diag_nodes(int64_t n_nodes, const uint8_t* __restrict__ interior,
                                                        const double* __restrict__ rho_new,
                                                        const double* __restrict__ rho_old,
                                                        const double* __restrict__ dtdg,
                                                        const double* __restrict__ dtMe,
                                                        const double* __restrict__ rG1, const double* __restrict__ rG2,
                                                        const double* __restrict__ dtrcg, int have_hist,
                                                        double c1, double c2, double* __restrict__ rG_out,
                                                        DiagAcc* acc) {
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    double v[4] = {0.0, 0.0, 0.0, 0.0};   // continuity, Gauss, rho, drift
    if (k < n_nodes) {
        if (!interior[k]) {
            rG_out[k] = 0.0;
        } else {
            const double rc = (rho_new[k] - rho_old[k]) - dtdg[k];
            const double rg = -dtMe[k] - rho_new[k];
            rG_out[k] = rg;
            v[0] = rc;
            v[1] = rg;
            v[2] = rho_new[k];
            if (have_hist) v[3] = (rg + c1 * rG1[k] + c2 * rG2[k]) - dtrcg[k];
        }
    }
    unsigned long long* const out[4] = {&acc->cont_max, &acc->gauss_max, &acc->rho_max, &acc->drift_max};
    block_max_abs<4>(v, out);
}

__global__ __launch_bounds__(kBlock) void k_divb(int64_t n_tets, const int32_t* __restrict__ tf,
                                                  const double* __restrict__ b, DiagAcc* acc) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    double v[1] = {0.0};
    if (t < n_tets) v[0] = b[tf[4 * t]] - b[tf[4 * t + 1]] + b[tf[4 * t + 2]] - b[tf[4 * t + 3]];
    unsigned long long* const out[1] = {&acc->divb_max};
    block_max_abs<1>(v, out);
}

__global__ __launch_bounds__(kBlock) void k_dot(int64_t n, RowGrid rg, const double* __restrict__ a,
                                                 const double* __restrict__ b, double* __restrict__ partial) {
    double v[1] = {0.0};
    for (int64_t lb = rg_first(rg), le = rg_end(rg); lb < le; lb += rg.g) {
        const int64_t i = lb * kBlock + threadIdx.x;
        if (i < n) v[0] += a[i] * b[i];
    }
    write_partials<1>(v, partial);
}

// Energy-norm step along a given direction d from e: x = e + theta d with
// theta = d.(b - A e) / d.A d = (b.d - e.(A d)) / (d.A d) (A symmetric), the minimiser of
// the A-norm error over the line, so x is never farther from the solution than e.
__global__ __launch_bounds__(kBlock) void k_line_dots(int64_t n_rows, RowGrid rg, const int64_t* __restrict__ sp,
                                                       const int32_t* __restrict__ col, const double* __restrict__ A,
                                                       const double* __restrict__ b, const double* __restrict__ e,
                                                       const double* __restrict__ d, double* __restrict__ partial) {
    double v[3] = {0.0, 0.0, 0.0};
    for (int64_t lb = rg_first(rg), le = rg_end(rg); lb < le; lb += rg.g) {
        const int64_t row = lb * kBlock + threadIdx.x;
        if (((row >> 6) << 6) >= n_rows) continue;
        const double ad = sell_row(sp, col, A, row, [&](int c) { return d[c]; });
        if (row < n_rows) {
            v[0] += b[row] * d[row];
            v[1] += e[row] * ad;
            v[2] += d[row] * ad;
        }
    }
    write_partials<3>(v, partial);
}

__global__ __launch_bounds__(kBlock) void k_line_theta(const double* __restrict__ partial, int n_src,
                                                        double* __restrict__ theta) {
    double t[3];
    read_partials<3>(partial, n_src, t);
    if (threadIdx.x == 0) theta[0] = (t[2] > 0.0 && isfinite(t[0] - t[1])) ? (t[0] - t[1]) / t[2] : 0.0;
}

__global__ __launch_bounds__(kBlock) void k_line_apply(int64_t n, const double* __restrict__ e,
                                                        const double* __restrict__ d,
                                                        const double* __restrict__ theta, double* __restrict__ x) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) x[i] = e[i] + theta[0] * d[i];
}

// Partial-buffer slots (each holds up to 3 values per workgroup of the largest grid).
constexpr size_t kSlot = 4 * kMaxGrid;
enum { SLOT_RHS = 0, SLOT_CG, SLOT_RESID, SLOT_DOT, SLOT_COUNT };
static_assert(4 * 3 * kCgSlots <= kSlot, "iteration slots fit one partial region");
static_assert(3 * 3 * kCgSlots + 2 * 3 * kBlockRows <= kSlot, "so do k_cg_iter<true>'s partials, behind them");

}  // namespace

size_t partial_buffer_doubles() { return SLOT_COUNT * kSlot; }

// ------------------------------------------------------------------------- launchers
void launch_fill(hipStream_t s, double* x, int64_t n, double v) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_fill, dim3(grid_1d(n, kBlock)), dim3(kBlock), 0, s, x, n, v);
}

void launch_read_out(hipStream_t s, const OutPieces& pieces, int n) {
    int64_t most = 1;
    for (int k = 0; k < n; ++k) most = std::max(most, pieces.p[k].n);
    hipLaunchKernelGGL(k_read_out, dim3((unsigned)std::min<int64_t>(grid_1d(most, kBlock), 256), (unsigned)n),
                       dim3(kBlock), 0, s, pieces);
}

void launch_axpby(hipStream_t s, double* y, const double* a, double alpha, const double* b, double beta, int64_t n) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_axpby, dim3(grid_1d(n, kBlock)), dim3(kBlock), 0, s, y, a, alpha, b, beta, n);
}

void launch_scale_A(hipStream_t s, const SellMatrix& shape, const int64_t* sp, const int32_t* col, const double* M,
                    const double* S, double* A, double* dinv, const uint8_t* bmask, double c, const double* K,
                    double cK) {
    const int64_t rows = shape.n_slices * kSell;
    hipLaunchKernelGGL(k_scale_A, dim3(grid_1d(rows, kBlock)), dim3(kBlock), 0, s, shape.n_rows, sp, col, M, S, A,
                       dinv, bmask, c, K, cK);
}

void launch_sell_spmv(hipStream_t s, int64_t n_rows, const int64_t* sp, const int32_t* col, const double* val,
                      const double* x, double* y) {
    hipLaunchKernelGGL(k_spmv, dim3(grid_1d(n_rows, kBlock)), dim3(kBlock), 0, s, n_rows, sp, col, val, x, y);
}

void launch_rhs(hipStream_t s, int64_t n_rows, const int64_t* sp, const int32_t* col, const double* M,
                const double* S, const double* e, const double* ep, const double* dg_new, const double* dg_old,
                const uint8_t* bmask, double dt2, double c1, double c2, const double* K, double k1, double k2,
                double* b, double* partial) {
    const RowGrid rg = row_grid(n_rows);
    if (K)
        hipLaunchKernelGGL(k_rhs<true>, dim3(rg.grid), dim3(kBlock), 0, s, n_rows, rg, sp, col, M, S, e, ep, dg_new,
                           dg_old, bmask, dt2, c1, c2, K, k1, k2, b, partial + SLOT_RHS * kSlot);
    else
        hipLaunchKernelGGL(k_rhs<false>, dim3(rg.grid), dim3(kBlock), 0, s, n_rows, rg, sp, col, M, S, e, ep, dg_new,
                           dg_old, bmask, dt2, c1, c2, K, k1, k2, b, partial + SLOT_RHS * kSlot);
}

void launch_mfem_rhs(hipStream_t s, int64_t n_rows, int64_t n_faces, const int64_t* sp, const int32_t* col,
                     const double* M, const double* S, const double* e, const double* ep, const double* dg_new,
                     const double* dg_old, const uint8_t* bmask, const int64_t* fsp, const int32_t* fcol,
                     const double* fval, const double* b1, double cb1, const double* b2, double cb2,
                     const int64_t* esp, const int32_t* einc, double* h, double dt, double a0, double a1, double s0,
                     double s1, double g0, double g1, double* bvec, double* partial) {
    hipLaunchKernelGGL(k_face_spmv, dim3(grid_1d((n_faces + 63) / 64 * 64, kBlock)), dim3(kBlock), 0, s, n_faces, fsp,
                       fcol, fval, b1, cb1, b2, cb2, h);
    const RowGrid rg = row_grid(n_rows);
    const MfemCoef k{a0, a1, s0, s1, g0, g1};
    hipLaunchKernelGGL(k_mfem_rhs, dim3(rg.grid), dim3(kBlock), 0, s, n_rows, rg, sp, col, M, S, e, ep, dg_new, dg_old,
                       bmask, esp, einc, h, dt, k, bvec, partial + SLOT_RHS * kSlot);
}

void launch_mfem_faraday(hipStream_t s, int64_t n_faces, const int32_t* face_edges, const double* b_base,
                         const double* e_n, const double* e_nm1, const double* e_np1, double dt, double cn, double cm,
                         double cp, double* b_new) {
    hipLaunchKernelGGL(k_mfem_faraday, dim3(grid_1d(n_faces, kBlock)), dim3(kBlock), 0, s, n_faces, face_edges, b_base,
                       e_n, e_nm1, e_np1, dt, cn, cm, cp, b_new);
}

void launch_warm(hipStream_t s, int mode, int64_t n, const double* e, const double* ep, const double* ep2, double* x) {
    hipLaunchKernelGGL(k_warm, dim3(grid_1d(n, kBlock)), dim3(kBlock), 0, s, mode, n, e, ep, ep2, x);
}

void launch_cg_init(hipStream_t s, int64_t n_rows, const int64_t* sp, const int32_t* col, const double* A,
                    const double* dinv, const double* b, const double* x, CgVec* v, double* partial, CgScalars* sc,
                    double tol, bool det) {
    const RowGrid rg = row_grid(n_rows, det ? kCgSlots : kMaxGrid);
    hipLaunchKernelGGL(k_cg_init_a, dim3(rg.grid), dim3(kBlock), 0, s, n_rows, rg, sp, col, A, dinv, b, x, v,
                       partial + SLOT_RHS * kSlot, (int)row_grid(n_rows).grid, partial + SLOT_CG * kSlot, sc, tol);
    hipLaunchKernelGGL(k_cg_init_b, dim3(rg.grid), dim3(kBlock), 0, s, n_rows, rg, sp, col, A, dinv, v,
                       partial + SLOT_CG * kSlot);
}

// One workgroup per block of kBlock rows (the iteration's partials do not grow with the
// grid), consecutive blocks on the same XCD.
inline RowGrid row_grid_full(int64_t n_rows) {
    RowGrid r;
    r.nb = (n_rows + kBlock - 1) / kBlock;
    r.per = (r.nb + 7) / 8;
    r.g = (int)std::max<int64_t>(1, r.per);
    r.grid = 8u * (unsigned)r.g;
    return r;
}

// At most max_grid workgroups over the row blocks (0: one each), consecutive blocks on the
// same XCD.
inline RowGrid block_grid(const BlockCols& bc, int max_grid = 0) {
    RowGrid r;
    r.nb = bc.nb;
    r.per = (r.nb + 7) / 8;
    r.g = (int)std::max<int64_t>(1, max_grid ? std::min<int64_t>(r.per, max_grid / 8) : r.per);
    r.grid = 8u * (unsigned)r.g;
    return r;
}

// Dynamic LDS of a staged vector: the block's own rows and its halo.
inline size_t staged_bytes(const BlockCols& bc, size_t value) { return value * (size_t)(kBlockRows + bc.stride); }

// Iteration i reads the interleaved state from buffer i & 1 and writes buffer (i + 1) & 1.
void launch_cg_iter(hipStream_t s, int i, int64_t n_rows, int n_max, const int64_t* sp, const int32_t* col,
                    const BlockCols& bc, const double* A, double* x, CgVec* const v[2], double* partial, CgScalars* sc,
                    bool det, bool twin) {
    const RowGrid rg = block_grid(bc, det && !twin ? kCgSlots : 0);
    const int a = i & 1, b = 1 - a;
    double* const slots = partial + SLOT_CG * kSlot;
    hipLaunchKernelGGL(twin ? k_cg_iter<true> : k_cg_iter<false>, dim3(rg.grid), dim3(kBlockRows),
                       staged_bytes(bc, sizeof(double)), s, n_rows, rg, i, twin ? n_max : INT32_MAX, sp, col, bc, A, x,
                       v[a], v[b], slots, slots + 3 * 3 * kCgSlots, sc);
}

int64_t cg_solve_boxes(const BlockCols& bc) { return bc.nb * (4 * kBlockRows + 12 * kSolveCopies); }

// One workgroup per CU: 197k rows on two per CU took 18.4 us per iteration, against 11.9 by
// k_cg_iter (129k rows, one per CU: 5.2 against 7.4).  Every halo column has a register
// (kHaloRegs) and every partial a thread.
bool cg_solve_fits(const BlockCols& bc, int n_cu) {
    if (bc.nb <= 0 || bc.nb > kBlockRows || bc.wide || bc.stride > kHaloRegs * kBlockRows) return false;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_cg_solve, kBlockRows,
                                                     staged_bytes(bc, sizeof(double))) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return per_cu > 0 && (int64_t)block_grid(bc).grid <= n_cu;
}

hipError_t launch_cg_solve(hipStream_t s, int64_t n_rows, int n_max, const int64_t* sp, const BlockCols& bc,
                           const double* A, const double* x, double* x_out, const CgVec* V,
                           unsigned long long* boxes, unsigned tag0, int polls, double* partial, CgScalars* sc) {
    RowGrid rg = block_grid(bc);
    BlockCols g = bc;
    const double* slots = partial + SLOT_CG * kSlot;
    unsigned box_bytes = (unsigned)(8 * cg_solve_boxes(bc));
    void* args[] = {&n_rows, &rg, &n_max, &sp, &g, &A, &x, &x_out, &V, &boxes, &box_bytes, &tag0, &polls, &slots, &sc};
    const hipError_t e = hipLaunchCooperativeKernel((const void*)k_cg_solve, dim3(rg.grid), dim3(kBlockRows), args,
                                                    (unsigned)staged_bytes(bc, sizeof(double)), s);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

namespace {
constexpr size_t kSolveLds = 152 * 1024;   // dynamic LDS of a workgroup alone on its CU

inline RowGrid solve_grid(const BlockCols& bc, int blocks) {
    RowGrid r;
    r.nb = (bc.nb + blocks - 1) / blocks;
    r.per = (r.nb + 7) / 8;
    r.g = (int)std::max<int64_t>(1, r.per);
    r.grid = 8u * (unsigned)r.g;
    return r;
}

// Dynamic LDS: what the phases use one after the other, and the state kept there.
inline size_t solve_shared(const BlockCols& bc, const SolveLists& l, int blocks, size_t value) {
    return value * std::max({blocks > 1 ? (size_t)0 : (size_t)(kBlockRows + bc.stride), (size_t)(8 * (l.stride + 1)),
                             (size_t)blocks * 4 * (kSolveNodes + 1)});
}
inline size_t solve_bytes(const BlockCols& bc, const SolveLists& l, int blocks, size_t value) {
    const size_t edges = (size_t)blocks * 2 * l.stride, rows = (size_t)blocks * kBlockRows;
    return solve_shared(bc, l, blocks, value) +
           (blocks > 1 ? edges * (12 + value) + (3 * rows + (size_t)blocks * bc.stride) * value : 0);
}

template <typename S>
const void* pcg_solve_kernel(int blocks) {
    return blocks == 1 ? (const void*)k_pcg_solve<S, 1> : (const void*)k_pcg_solve<S, 2>;
}

// One workgroup per CU with one or two row blocks: with four (FP32, 463k rows) the matrix and
// state spilled 740 bytes per lane and an iteration took 50 us, against 27 by the kernels;
// with two they lose on no mesh that fits (figures at k_pcg_solve).
template <typename S>
bool pcg_solve_resident(const BlockCols& bc, const SolveLists& l, int blocks, int n_cu) {
    const RowGrid rg = solve_grid(bc, blocks);
    if (l.n_slices > 2 * blocks * rg.nb || rg.nb > kBlockRows || (int64_t)rg.grid > n_cu) return false;
    int per_cu = 0;
    const size_t lds = solve_bytes(bc, l, blocks, sizeof(S));
    if (lds > kSolveLds || hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, pcg_solve_kernel<S>(blocks), kBlockRows,
                                                                        lds) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return per_cu > 0;
}
}  // namespace

template <typename S>
int pcg_solve_blocks(const BlockCols& bc, const SolveLists& l, int n_cu) {
    if (l.n_slices == 0 || bc.nb <= 0 || bc.wide || bc.stride > kHaloRegs * kBlockRows) return 0;
    for (int blocks : {1, 2})
        if (pcg_solve_resident<S>(bc, l, blocks, n_cu)) return blocks;
    return 0;
}

template <typename S>
int64_t pcg_solve_boxes(const BlockCols& bc, const SolveLists& l, int64_t n_rows, int64_t n_aux, int blocks) {
    return (int64_t)(sizeof(S) / 4) * (2 * n_rows + 4 * n_aux + 4 * l.n_slices) +
           6 * kSolveCopies * solve_grid(bc, blocks).nb;
}

template <typename S, typename S2>
hipError_t launch_pcg_solve(hipStream_t s, int blocks, int64_t n_rows, int n_max, const int64_t* sp,
                            const BlockCols& bc, const S* A, const S* dinv, const S* x, S* x_out, const S2* zp0,
                            const S* r, const AuxSpace& g, const SolveLists& l, unsigned long long* boxes, unsigned tag0,
                            int polls, double* partial, CgScalars* sc) {
    RowGrid rg = solve_grid(bc, blocks);
    BlockCols b = bc;
    AuxSpace a = g;
    SolveLists ll = l;
    const double* slots = partial + SLOT_CG * kSlot + (size_t)3 * 3 * kCgSlots;   // reduction -1: buffer 3 of 4
    unsigned box_bytes = (unsigned)(8 * pcg_solve_boxes<S>(bc, l, n_rows, g.n_aux, blocks));
    unsigned shared_bytes = (unsigned)solve_shared(bc, l, blocks, sizeof(S));
    void* args[] = {&n_rows, &rg, &n_max, &sp,    &b,         &A,            &dinv, &x,     &x_out, &zp0,
                    &r,      &a,  &ll,    &boxes, &box_bytes, &shared_bytes, &tag0, &polls, &slots, &sc};
    const hipError_t e = hipLaunchCooperativeKernel(pcg_solve_kernel<S>(blocks), dim3(rg.grid), dim3(kBlockRows), args,
                                                    (unsigned)solve_bytes(bc, l, blocks, sizeof(S)), s);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

template int pcg_solve_blocks<double>(const BlockCols&, const SolveLists&, int);
template int pcg_solve_blocks<float>(const BlockCols&, const SolveLists&, int);
template int64_t pcg_solve_boxes<double>(const BlockCols&, const SolveLists&, int64_t, int64_t, int);
template int64_t pcg_solve_boxes<float>(const BlockCols&, const SolveLists&, int64_t, int64_t, int);
template hipError_t launch_pcg_solve<double, double2>(hipStream_t, int, int64_t, int, const int64_t*, const BlockCols&,
                                                      const double*, const double*, const double*, double*,
                                                      const double2*, const double*, const AuxSpace&, const SolveLists&,
                                                      unsigned long long*, unsigned, int, double*, CgScalars*);
template hipError_t launch_pcg_solve<float, float2>(hipStream_t, int, int64_t, int, const int64_t*, const BlockCols&,
                                                    const float*, const float*, const float*, float*, const float2*,
                                                    const float*, const AuxSpace&, const SolveLists&, unsigned long long*, unsigned, int,
                                                    double*, CgScalars*);

// One workgroup per slice of 64 auxiliary nodes, consecutive slices on the same XCD.
inline RowGrid node_grid(int64_t n_aux) {
    RowGrid r;
    r.nb = (n_aux + 63) / 64;
    r.per = (r.nb + 7) / 8;
    r.g = (int)std::max<int64_t>(1, r.per);
    r.grid = 8u * (unsigned)r.g;
    return r;
}

void launch_aux_scale(hipStream_t s, const AuxSpace& g, const int64_t* sp, const int32_t* col, const double* A) {
    if (g.n_aux <= 0) return;
    const int64_t n8 = 4 * ((g.n_aux + 7) / 8), n64 = 4 * ((g.n_aux + 63) / 64);
    hipLaunchKernelGGL(k_aux_scale, dim3(grid_1d(g.n_aux, kBlock)), dim3(kBlock), 0, s, g, sp, col, A);
    hipLaunchKernelGGL(k_fill, dim3(grid_1d(n8, kBlock)), dim3(kBlock), 0, s, reinterpret_cast<double*>(g.scale8), n8,
                       0.0);
    hipLaunchKernelGGL(k_fill, dim3(grid_1d(n64, kBlock)), dim3(kBlock), 0, s, reinterpret_cast<double*>(g.scale64),
                       n64, 0.0);
    for (int L = 0; L < kAuxFarLevels; ++L) {
        const int64_t nf = 4 * aux_far_count(g.n_aux, L);
        hipLaunchKernelGGL(k_fill, dim3(grid_1d(nf, kBlock)), dim3(kBlock), 0, s,
                           reinterpret_cast<double*>(g.far_scale[L]), nf, 0.0);
    }
    hipLaunchKernelGGL(k_aux_coarse, dim3(grid_1d(g.n_aux, kBlock)), dim3(kBlock), 0, s, g, sp, col, A);
    hipLaunchKernelGGL(k_invert_pos, dim3(grid_1d(n8, kBlock)), dim3(kBlock), 0, s, reinterpret_cast<double*>(g.scale8),
                       n8);
    hipLaunchKernelGGL(k_invert_pos, dim3(grid_1d(n64, kBlock)), dim3(kBlock), 0, s,
                       reinterpret_cast<double*>(g.scale64), n64);
    for (int L = 0; L < kAuxFarLevels; ++L) {
        const int64_t nf = 4 * aux_far_count(g.n_aux, L);
        hipLaunchKernelGGL(k_invert_pos, dim3(grid_1d(nf, kBlock)), dim3(kBlock), 0, s,
                           reinterpret_cast<double*>(g.far_scale[L]), nf);
    }
}

namespace {
template <typename S>
void product(hipStream_t s, int i, int64_t n_rows, const int64_t* sp, const int32_t* col, const BlockCols& bc,
             const S* A, const typename Vec<S>::t2* zp, S* Q, double* slots, CgScalars* sc, const AuxSpace& g) {
    const RowGrid rg = block_grid(bc);
    hipLaunchKernelGGL(k_pcg_q<S>, dim3(rg.grid), dim3(kBlockRows), staged_bytes(bc, sizeof(S)), s, n_rows, rg, i, sp,
                       col, bc, A, zp, Q, slots, sc, g);
}

template <typename S>
void pcg_start(hipStream_t s, int64_t n_rows, const int64_t* sp, const int32_t* col, const S* A, const S* dinv,
               const double* b, S* x, bool zero_x, const AuxSpace& g, typename Vec<S>::t2* zp0, S* R, S* Q,
               const double* part_b, double* slots, CgScalars* sc, double tol) {
    const RowGrid rg = row_grid(n_rows);
    hipLaunchKernelGGL(k_pcg_init<S>, dim3(rg.grid), dim3(kBlock), 0, s, n_rows, rg, sp, col, A, b, x, zero_x, R, Q,
                       part_b, slots, sc, tol, g);
    const RowGrid ng = node_grid(g.n_aux);
    hipLaunchKernelGGL(k_pcg_nodes<S>, dim3(ng.grid), dim3(kBlock), 0, s, ng, -1, g, (const S*)R, (const S*)Q, slots,
                       sc);
    if (g.n_far > 0)
        hipLaunchKernelGGL(k_pcg_fold<S>, dim3(grid_1d(g.n_aux, kBlock)), dim3(kBlock), 0, s, g, sc);
    constexpr int kR = update_rows<S>();
    const RowGrid ug = row_grid_full((n_rows + kR - 1) / kR);
    hipLaunchKernelGGL((k_pcg_update<S, kR>), dim3(ug.grid), dim3(kBlock), 0, s, n_rows, ug, -1, g, dinv, x,
                       (const typename Vec<S>::t2*)zp0, zp0, R, (const S*)Q, slots, sc);
}

template <typename S>
void pcg_iter(hipStream_t s, int i, int64_t n_rows, const int64_t* sp, const int32_t* col, const BlockCols& bc,
              const S* A, const S* dinv, S* x, const AuxSpace& g, typename Vec<S>::t2* const zp[2], S* R, S* Q,
              double* slots, CgScalars* sc) {
    const RowGrid ng = node_grid(g.n_aux);
    const int a = i & 1, b = 1 - a;
    product<S>(s, i, n_rows, sp, col, bc, A, zp[a], Q, slots, sc, g);
    hipLaunchKernelGGL(k_pcg_nodes<S>, dim3(ng.grid), dim3(kBlock), 0, s, ng, i, g, (const S*)R, (const S*)Q, slots,
                       sc);
    if (g.n_far > 0)
        hipLaunchKernelGGL(k_pcg_fold<S>, dim3(grid_1d(g.n_aux, kBlock)), dim3(kBlock), 0, s, g, sc);
    constexpr int kR = update_rows<S>();
    const RowGrid ug = row_grid_full((n_rows + kR - 1) / kR);
    hipLaunchKernelGGL((k_pcg_update<S, kR>), dim3(ug.grid), dim3(kBlock), 0, s, n_rows, ug, i, g, dinv, x,
                       (const typename Vec<S>::t2*)zp[a], zp[b], R, (const S*)Q, slots, sc);
}
}  // namespace

// The start: r = b - A x, then z = B r and the dots (r, z), (r, r) as reduction -1.
void launch_pcg_init(hipStream_t s, int64_t n_rows, const int64_t* sp, const int32_t* col, const double* A,
                     const double* dinv, const double* b, const double* x, const AuxSpace& g, double2* zp0,
                     double2* rq, double* partial, CgScalars* sc, double tol) {
    double* R = reinterpret_cast<double*>(rq);
    pcg_start<double>(s, n_rows, sp, col, A, dinv, b, const_cast<double*>(x), false, g, zp0, R, R + n_rows,
                      partial + SLOT_RHS * kSlot, partial + SLOT_CG * kSlot, sc, tol);
}

// Iteration i: (z, p) pairs read from buffer i & 1, the new pair written to (i + 1) & 1;
// r in the first n_rows doubles of rq, q in the next n_rows.
void launch_pcg_iter(hipStream_t s, int i, int64_t n_rows, const int64_t* sp, const int32_t* col,
                     const BlockCols& bc, const double* A, const double* dinv, double* x, const AuxSpace& g,
                     double2* const zp[2], double2* rq, double* partial, CgScalars* sc) {
    double* R = reinterpret_cast<double*>(rq);
    pcg_iter<double>(s, i, n_rows, sp, col, bc, A, dinv, x, g, zp, R, R + n_rows, partial + SLOT_CG * kSlot, sc);
}

// The inner solve of the mixed-precision form: A d = r in FP32 from d = 0, r the FP64
// true residual that launch_cg_resid left in r_true (its norm from that kernel's partials).
void launch_pcg_init_f32(hipStream_t s, int64_t n_rows, const int64_t* sp, const int32_t* col,
                         const float* dinv32, const double* r_true, float* d, const AuxSpace& g, float2* zp0, float* rq,
                         double* partial, CgScalars* sc, double tol) {
    pcg_start<float>(s, n_rows, sp, col, nullptr, dinv32, r_true, d, true, g, zp0, rq, rq + n_rows,
                     partial + SLOT_RESID * kSlot, partial + SLOT_CG * kSlot, sc, tol);
}

void launch_pcg_iter_f32(hipStream_t s, int i, int64_t n_rows, const int64_t* sp, const int32_t* col,
                         const BlockCols& bc, const float* A32, const float* dinv32, float* d, const AuxSpace& g,
                         float2* const zp[2], float* rq, double* partial, CgScalars* sc) {
    pcg_iter<float>(s, i, n_rows, sp, col, bc, A32, dinv32, d, g, zp, rq, rq + n_rows, partial + SLOT_CG * kSlot, sc);
}

void launch_block_count(hipStream_t s, const BlockCols& g, const int64_t* sp, const int32_t* col, int32_t* cnt) {
    if (g.nb > 0)
        hipLaunchKernelGGL(k_block_cols<false>, dim3((unsigned)g.nb), dim3(kBlock), 0, s, g, sp, col, cnt, nullptr,
                           nullptr);
}

void launch_block_fill(hipStream_t s, const BlockCols& g, const int64_t* sp, const int32_t* col, int32_t* halo,
                       uint16_t* lcol) {
    if (g.nb > 0)
        hipLaunchKernelGGL(k_block_cols<true>, dim3((unsigned)g.nb), dim3(kBlock), 0, s, g, sp, col, nullptr, halo, lcol);
}

// FP32 copies of the operator for the inner solves: A (in the pair layout), D^-1, and the
// auxiliary space's inverse diagonals at every level.
void launch_operator_f32(hipStream_t s, int64_t n_slices, const int64_t* sp, const double* A, float* A32,
                         int64_t n_rows, const double* dinv, float* dinv32, const AuxSpace& g) {
    auto cvt = [&](const void* a, void* b, int64_t n) {
        if (n > 0)
            hipLaunchKernelGGL(k_to_f32, dim3(grid_1d(n, kBlock)), dim3(kBlock), 0, s,
                               reinterpret_cast<const double*>(a), reinterpret_cast<float*>(b), n);
    };
    hipLaunchKernelGGL(k_pack_f32, dim3(grid_1d(64 * n_slices, kBlock)), dim3(kBlock), 0, s, n_slices, sp, A, A32);
    cvt(dinv, dinv32, n_rows);
    cvt(g.scale, g.scale_f, 4 * g.n_aux);
    cvt(g.scale8, g.scale8_f, 4 * ((g.n_aux + 7) / 8));
    cvt(g.scale64, g.scale64_f, 4 * ((g.n_aux + 63) / 64));
    for (int L = 0; L < kAuxFarLevels; ++L) cvt(g.far_scale[L], g.far_scale_f[L], 4 * aux_far_count(g.n_aux, L));
}

void launch_pcg_rhs_norm(hipStream_t s, int64_t n_rows, double* partial, CgScalars* sc, double tol) {
    hipLaunchKernelGGL(k_rhs_norm, dim3(1), dim3(kBlock), 0, s, partial + SLOT_RHS * kSlot, (int)row_grid(n_rows).grid,
                       sc, tol);
}

void launch_add_f32(hipStream_t s, double* x, const float* d, int64_t n) {
    if (n > 0) hipLaunchKernelGGL(k_add_f32, dim3(grid_1d(n, kBlock)), dim3(kBlock), 0, s, x, d, n);
}

void launch_pcg_rr0(hipStream_t s, double* partial, CgScalars* sc) {
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(kBlock), 0, s, partial + SLOT_CG * kSlot + 3 * 3 * kCgSlots + kCgSlots,
                       kCgSlots, &sc->rr0);
}

void launch_cg_rr0(hipStream_t s, int64_t n_rows, double* partial, CgScalars* sc) {
    (void)n_rows;
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(kBlock), 0, s, partial + SLOT_CG * kSlot + 2 * kCgSlots, kCgSlots,
                       &sc->rr0);
}

void launch_cg_resid(hipStream_t s, int64_t n_rows, const int64_t* sp, const int32_t* col, const double* A,
                     const double* b, double* x, double* r_true, double* partial, CgScalars* sc) {
    hipLaunchKernelGGL(k_zero_if_b_zero, dim3(grid_1d(n_rows, kBlock)), dim3(kBlock), 0, s, x, n_rows, sc);
    const RowGrid rg = row_grid(n_rows);
    hipLaunchKernelGGL(k_cg_resid, dim3(rg.grid), dim3(kBlock), 0, s, n_rows, rg, sp, col, A, b, x, r_true,
                       partial + SLOT_RESID * kSlot);
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(kBlock), 0, s, partial + SLOT_RESID * kSlot, (int)rg.grid,
                       &sc->rr_true);
}

void launch_faraday(hipStream_t s, int64_t n_faces, const int32_t* face_edges, const double* b_old,
                    const double* e_new, const double* e_old, double dt, double gamma, double* b_new) {
    if (n_faces <= 0) return;
    hipLaunchKernelGGL(k_faraday, dim3(grid_1d(n_faces, kBlock)), dim3(kBlock), 0, s, n_faces, face_edges, b_old,
                       e_new, e_old, dt, gamma, b_new);
}

void launch_DT(hipStream_t s, int64_t n_edges, const int32_t* edges, const double* v, double* out_nodes) {
    hipLaunchKernelGGL(k_DT, dim3(grid_1d(n_edges, kBlock)), dim3(kBlock), 0, s, n_edges, edges, v, out_nodes);
}

void launch_diag_nodes(hipStream_t s, int64_t n_nodes, const uint8_t* interior_node, const double* rho_new,
                       const double* rho_old, const double* dtdg, const double* dtMe, const double* rG1,
                       const double* rG2, const double* dtrcg, int have_hist, double c1, double c2, double* rG_out,
                       DiagAcc* acc) {
    hipLaunchKernelGGL(k_diag_nodes, dim3(grid_1d(n_nodes, kBlock)), dim3(kBlock), 0, s, n_nodes, interior_node,
                       rho_new, rho_old, dtdg, dtMe, rG1, rG2, dtrcg, have_hist, c1, c2, rG_out, acc);
}

void launch_divb(hipStream_t s, int64_t n_tets, const int32_t* tet_faces, const double* b, DiagAcc* acc) {
    hipLaunchKernelGGL(k_divb, dim3(grid_1d(n_tets, kBlock)), dim3(kBlock), 0, s, n_tets, tet_faces, b, acc);
}

void launch_line_start(hipStream_t s, int64_t n_rows, const int64_t* sp, const int32_t* col, const double* A,
                       const double* b, const double* e, const double* d, double* partial, double* theta, double* x) {
    const RowGrid rg = row_grid(n_rows);
    hipLaunchKernelGGL(k_line_dots, dim3(rg.grid), dim3(kBlock), 0, s, n_rows, rg, sp, col, A, b, e, d,
                       partial + SLOT_DOT * kSlot);
    hipLaunchKernelGGL(k_line_theta, dim3(1), dim3(kBlock), 0, s, partial + SLOT_DOT * kSlot, (int)rg.grid, theta);
    hipLaunchKernelGGL(k_line_apply, dim3(grid_1d(n_rows, kBlock)), dim3(kBlock), 0, s, n_rows, e, d, theta, x);
}

void launch_dot(hipStream_t s, int64_t n, const double* a, const double* b, double* partial, double* out) {
    const RowGrid rg = row_grid(n);
    hipLaunchKernelGGL(k_dot, dim3(rg.grid), dim3(kBlock), 0, s, n, rg, a, b, partial + SLOT_DOT * kSlot);
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(kBlock), 0, s, partial + SLOT_DOT * kSlot, (int)rg.grid, out);
}

}  // namespace fepic
