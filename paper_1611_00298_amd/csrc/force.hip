// force.hip -- EOFA pseudofermion force (eq. (3.2)) and the MD link update.
//
// For a link U_mu(x) the variation of S = phi^dag M_EOFA phi is
//   k chi_L^dag g5 R5 (dD_w) chi_L - k chi_R^dag g5 R5 (dD_w) chi_R.
// With eta = g5 R5 chi and B[chi] = sum_{s,spin} chi_s(x) (x) ((1+gamma_mu) eta_s(x+mu))^dag
// the complex gradient (dS = Re tr(G^dag dU)) is G = -sigma k (B[chi_L] - B[chi_R]),
// and the su(3) force F = sum_a T^a d^a S is (1/4) TA(-i W) with
// W = sigma k (U B^dag - B U^dag), B = B[chi_L] - B[chi_R], sigma the
// boundary sign of the link.  Because (1+gamma_mu) has rank two,
// B = sum_{s} sum_{j=0,1} h_j (x) g_j^dag with h = chi_up + A_mu chi_lo at x
// and g = chi_up - A_mu chi_lo at (x+mu, Ls-1-s) (the minus sign is gamma_5).
// FP64 throughout; one work-item per link, chi in the natural layout.
#include "internal.h"
#include <type_traits>

namespace eofa {

struct cplx {
    double r, i;
};
__device__ __forceinline__ cplx cmul(cplx a, cplx b) { return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r}; }
__device__ __forceinline__ cplx cmulc(cplx a, cplx b) { return {a.r * b.r + a.i * b.i, a.i * b.r - a.r * b.i}; }  // a conj(b)

// (A_mu v_lo)_j for the chiral-basis block A_mu of gamma_mu (see dslash.hip)
__device__ __forceinline__ void amul(int mu, cplx v2, cplx v3, cplx& o0, cplx& o1) {
    switch (mu) {
    case 0: o0 = {v3.i, -v3.r}; o1 = {v2.i, -v2.r}; break;     // -i v3, -i v2
    case 1: o0 = {-v3.r, -v3.i}; o1 = {v2.r, v2.i}; break;     // -v3, v2
    case 2: o0 = {v2.i, -v2.r}; o1 = {-v3.i, v3.r}; break;     // -i v2, i v3
    default: o0 = v2; o1 = v3; break;                          // v2, v3
    }
}

// F and G of one link from B = B[chi_L] - B[chi_R] and the link U (natural
// layout entries, row major), sigma the boundary sign of the link:
//   W = sigma k (U B^dag - B U^dag),  F = 1/4 TA(-i W),  G = -sigma k B.
__device__ __forceinline__ void force_from_B(const cplx (&B)[9], const double2* __restrict__ Ul, double sigma, double k,
                             double2* __restrict__ Fl, double2* __restrict__ Gl) {
    cplx u[9];
    for (int q = 0; q < 9; ++q) u[q] = {Ul[q].x, Ul[q].y};
    cplx Y[9];   // Y = -i W
    for (int x = 0; x < 3; ++x)
        for (int y = 0; y < 3; ++y) {
            cplx w = {0.0, 0.0};
            for (int q = 0; q < 3; ++q) {
                const cplx t1 = cmulc(u[3 * x + q], B[3 * y + q]);   // U_xq conj(B_yq)
                const cplx t2 = cmulc(B[3 * x + q], u[3 * y + q]);   // B_xq conj(U_yq)
                w.r += t1.r - t2.r;
                w.i += t1.i - t2.i;
            }
            w.r *= sigma * k;
            w.i *= sigma * k;
            Y[3 * x + y] = {w.i, -w.r};
        }
    // F = 1/4 [ (Y + Y^dag)/2 - tr(Y + Y^dag)/6 ]
    const double tr = (Y[0].r + Y[4].r + Y[8].r) / 3.0;
    for (int x = 0; x < 3; ++x)
        for (int y = 0; y < 3; ++y) {
            const cplx a = Y[3 * x + y], b = Y[3 * y + x];
            double re = 0.5 * (a.r + b.r), im = 0.5 * (a.i - b.i);
            if (x == y) re -= tr;
            Fl[3 * x + y] = make_double2(0.25 * re, 0.25 * im);
        }
    if (Gl) {
        const double f = -sigma * k;
        for (int q = 0; q < 9; ++q) Gl[q] = make_double2(f * B[q].r, f * B[q].i);
    }
}

// A workgroup owns a 4D tile of 64 sites (two extents of 4 and two of 2) and
// all four directions: wavefront mu takes direction mu, its lanes the sites,
// so the sum over s stays in each work-item's registers.  chi is read in the
// natural layout, where a 4D site's spinor of one slice is 192 contiguous
// bytes.  Per step the workgroup stages two slices, s and Ls-1-s, of the
// tile and its four forward faces in LDS and forms both products of the pair
// (own slice s with the neighbours' Ls-1-s, and the other way round).
// A slice pair costs 2.5 spinor reads per site (own and faces) where a gather
// per direction costs 5, and the next step's words are in registers while a
// step computes.  Bound by memory: at 24^3x64, Ls = 24 it takes 3.10 ms for
// 8.7 GB of operands (about 1.5 times that from beyond L2); a per-5D-site
// gather in the device layout took 4.10 ms after two layout passes of 1.98 ms.
// At 16^3x32, Ls = 16 with G: 0.33 ms against 0.86 ms.
// Slots: 64 own sites, then the faces x+mu of the four directions; a slot
// beyond the lattice (ragged tiles) holds the site it wraps to.
constexpr int FT_SITES = 64;
constexpr int FT_SLOTS = FT_SITES + 16 + 16 + 32 + 32;
constexpr int FT_STR = FT_SLOTS + 1;            // odd: the records' 12 words spread over the banks
constexpr int FT_CHUNKS = FT_SLOTS * 12;        // 16-byte words of one staged slice
constexpr int FT_LOADS = (FT_CHUNKS + 255) / 256;

struct ForceTile {
    int lg[4];   // log2 of the tile extents (1 or 2)
    int n[4];    // tiles along each direction
    int tiles;
    int split;   // > 0: ranges of slice pairs per system, each a workgroup's
};

// origin of tile r, and a lane's site in it (own); false: beyond the lattice
__device__ __forceinline__ bool tile_site(const ForceTile& ft, const Geo& g, int r, int lane, int (&o)[4], int (&own)[4]) {
    bool active = true;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        o[d] = (r % ft.n[d]) << ft.lg[d];
        r /= ft.n[d];
        own[d] = lane & ((1 << ft.lg[d]) - 1);
        lane >>= ft.lg[d];
        active = active && o[d] + own[d] < g.L[d];
    }
    return active;
}

// acc += sum_j h_j (x) g_j^dag, h_j of the spinor at p and g_j of the one at q.
// The slice's four products are summed before they join the accumulator: 2 Ls
// roundings at the size of the whole sum would be 8 Ls, and an error 2.2 times
// as large at Ls = 16, with each product added to the accumulator by itself.
template <int MU>
__device__ __forceinline__ void force_pair(const d2v* __restrict__ p, const d2v* __restrict__ q,
                                           cplx (&acc)[9]) {
    cplx h[2][3], gg[2][3];
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
        const d2v a0 = p[cc * FT_STR], a1 = p[(3 + cc) * FT_STR];
        const d2v a2 = p[(6 + cc) * FT_STR], a3 = p[(9 + cc) * FT_STR];
        const d2v b0 = q[cc * FT_STR], b1 = q[(3 + cc) * FT_STR];
        const d2v b2 = q[(6 + cc) * FT_STR], b3 = q[(9 + cc) * FT_STR];
        cplx p0, p1, q0, q1;
        amul(MU, {a2.x, a2.y}, {a3.x, a3.y}, p0, p1);
        amul(MU, {b2.x, b2.y}, {b3.x, b3.y}, q0, q1);
        h[0][cc] = {a0.x + p0.r, a0.y + p0.i};
        h[1][cc] = {a1.x + p1.r, a1.y + p1.i};
        gg[0][cc] = {b0.x - q0.r, b0.y - q0.i};
        gg[1][cc] = {b1.x - q1.r, b1.y - q1.i};
    }
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int y = 0; y < 3; ++y) {
            const cplx u0 = h[0][x], v0 = gg[0][y], u1 = h[1][x], v1 = gg[1][y];
            cplx& o = acc[3 * x + y];
            o.r += fmadd(u1.r, v1.r, fmadd(u1.i, v1.i, fmadd(u0.r, v0.r, u0.i * v0.i)));
            o.i += fmadd(u1.i, v1.r, fmadd(-u1.r, v1.i, fmadd(u0.i, v0.r, -u0.r * v0.i)));
        }
}

// Small lattices have few tiles: with SPLIT, a workgroup takes one system and
// one of ft.split ranges of its slice pairs and leaves its sums in part,
// [2 split][tile][9][256]; k_force_finish adds them up.
template <bool SPLIT>
__global__ void __launch_bounds__(256, 2) k_force(const double2* __restrict__ chiL, const double2* __restrict__ chiR,
                                                  const double2* __restrict__ U, double k, double2* __restrict__ F,
                                                  double2* __restrict__ G, Geo g, ForceTile ft, double2* __restrict__ part) {
    __shared__ d2v tile[2][12 * FT_STR];
    __shared__ int nat[FT_SLOTS];   // natural site index of each slot
    const int tid = threadIdx.x, mu = tid >> 6, lane = tid & 63;
    const int blk = xcd_block(gridDim.x), rng = SPLIT ? blk / ft.tiles : 0;
    int o[4], own[4];   // tile origin, this lane's site
    const bool active = tile_site(ft, g, blk - rng * ft.tiles, lane, o, own);
    // first slot of each face
    int face[4];
    face[0] = FT_SITES;
#pragma unroll
    for (int d = 1; d < 4; ++d) face[d] = face[d - 1] + (FT_SITES >> ft.lg[d - 1]);
    if (tid < FT_SLOTS) {
        int fd = -1, r = tid;   // face direction (-1: own site) and index within it
#pragma unroll
        for (int d = 0; d < 4; ++d)
            if (tid >= face[d]) { fd = d; r = tid - face[d]; }
        int i = 0, stride = 1;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            int c = 1 << ft.lg[d];
            if (d != fd) { c = r & (c - 1); r >>= ft.lg[d]; }
            i += ((o[d] + c) % g.L[d]) * stride;
            stride *= g.L[d];
        }
        nat[tid] = i;
    }
    // the slot of this lane's neighbour along mu
    int nb = 0, sh = 0, step = 1;
    bool inside = true;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        if (d == mu) inside = own[d] + 1 < (1 << ft.lg[d]);
        else { nb |= own[d] << sh; sh += ft.lg[d]; }
        if (d < mu) step <<= ft.lg[d];
    }
    nb = inside ? lane + step : nb + (mu == 0 ? face[0] : mu == 1 ? face[1] : mu == 2 ? face[2] : face[3]);
    __syncthreads();
    // staging: word c of slot j by work-item (12 j + c) mod 256; the work-items past the end repeat the last word
    uint32_t src[FT_LOADS];
    int dst[FT_LOADS];
#pragma unroll
    for (int u = 0; u < FT_LOADS; ++u) {
        const int e = min(tid + 256 * u, FT_CHUNKS - 1), j = e / 12, c = e - 12 * j;
        src[u] = (uint32_t)nat[j] * 12u + (uint32_t)c;
        dst[u] = c * FT_STR + j;
    }
    const int Ls = g.Ls, half = (Ls + 1) / 2;
    const size_t slice = (size_t)g.V * 12;
    d2v va[FT_LOADS], vb[FT_LOADS];
    auto fetch = [&](int it) __attribute__((always_inline)) {   // step it: system it / half, slices q and Ls-1-q
        const double2* chi = it < half ? chiL : chiR;
        const int q = it < half ? it : it - half;
        const d2v* a = reinterpret_cast<const d2v*>(chi + (size_t)q * slice);
        const d2v* b = reinterpret_cast<const d2v*>(chi + (size_t)(Ls - 1 - q) * slice);
#pragma unroll
        for (int u = 0; u < FT_LOADS; ++u) va[u] = a[src[u]];
#pragma unroll
        for (int u = 0; u < FT_LOADS; ++u) vb[u] = b[src[u]];
    };
    cplx acc[9], accL[9];   // this system's sum, and chi_L's once it is complete
#pragma unroll
    for (int q = 0; q < 9; ++q) acc[q] = {0.0, 0.0};
    int it0 = 0, it1 = 2 * half;
    if constexpr (SPLIT) {
        const int sys = rng >= ft.split, j = rng - sys * ft.split;
        it0 = sys * half + half * j / ft.split;
        it1 = sys * half + half * (j + 1) / ft.split;
    }
    fetch(it0);
#pragma unroll 1
    for (int it = it0; it < it1; ++it) {
        __syncthreads();   // the previous step's slices are read
#pragma unroll
        for (int u = 0; u < FT_LOADS; ++u) {
            tile[0][dst[u]] = va[u];
            tile[1][dst[u]] = vb[u];
        }
        __syncthreads();
        if (it + 1 < it1) fetch(it + 1);   // in flight while this step computes
        const int q = it < half ? it : it - half;
        const int n = 2 * q + 1 == Ls ? 1 : 2;   // the middle slice of an odd Ls pairs with itself
        auto pair = [&](auto m) __attribute__((always_inline)) {
            force_pair<decltype(m)::value>(tile[0] + lane, tile[1] + nb, acc);
            if (n == 2) force_pair<decltype(m)::value>(tile[1] + lane, tile[0] + nb, acc);
        };
        switch (mu) {   // once per pair: 8^3x32, Ls = 64 169 -> 162 us against a switch per slice
        case 0: pair(std::integral_constant<int, 0>()); break;
        case 1: pair(std::integral_constant<int, 1>()); break;
        case 2: pair(std::integral_constant<int, 2>()); break;
        default: pair(std::integral_constant<int, 3>()); break;
        }
        if (!SPLIT && it == half - 1) {
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                accL[e] = acc[e];
                acc[e] = {0.0, 0.0};
            }
        }
    }
    if constexpr (SPLIT) {
        double2* dst2 = part + (size_t)blk * 9 * 256 + tid;
#pragma unroll
        for (int e = 0; e < 9; ++e) dst2[e * 256] = make_double2(acc[e].r, acc[e].i);
        return;
    }
#pragma unroll
    for (int e = 0; e < 9; ++e) acc[e] = {accL[e].r - acc[e].r, accL[e].i - acc[e].i};
    if (active) {
        const double sigma = (mu == 3 && g.aperiodic && o[3] + own[3] == g.L[3] - 1) ? -1.0 : 1.0;
        const size_t l = ((size_t)mu * g.V + nat[lane]) * 9;
        force_from_B(acc, U + l, sigma, k, F + l, G ? G + l : nullptr);
    }
}

// F and G from the sums of k_force<true>, one tile per workgroup, in the order of the ranges
__global__ void __launch_bounds__(256) k_force_finish(const double2* __restrict__ part, const double2* __restrict__ U,
                                                      double k, double2* __restrict__ F, double2* __restrict__ G, Geo g,
                                                      ForceTile ft) {
    const int tid = threadIdx.x, mu = tid >> 6;
    int o[4], own[4];
    if (!tile_site(ft, g, blockIdx.x, tid & 63, o, own)) return;
    cplx B[2][9];
#pragma unroll
    for (int sys = 0; sys < 2; ++sys) {
#pragma unroll
        for (int e = 0; e < 9; ++e) B[sys][e] = {0.0, 0.0};
        for (int j = 0; j < ft.split; ++j) {
            const double2* p = part + ((size_t)(sys * ft.split + j) * ft.tiles + blockIdx.x) * 9 * 256 + tid;
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                const double2 v = p[e * 256];
                B[sys][e].r += v.x;
                B[sys][e].i += v.y;
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 9; ++e) B[0][e] = {B[0][e].r - B[1][e].r, B[0][e].i - B[1][e].i};
    int i = 0, stride = 1;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        i += (o[d] + own[d]) * stride;
        stride *= g.L[d];
    }
    const double sigma = (mu == 3 && g.aperiodic && o[3] + own[3] == g.L[3] - 1) ? -1.0 : 1.0;
    const size_t l = ((size_t)mu * g.V + i) * 9;
    force_from_B(B[0], U + l, sigma, k, F + l, G ? G + l : nullptr);
}

// ---------------------------------------------------------------------------
// MD: P <- P - dt_p F ; U <- exp(i dt_u P) U ; partial sum of tr P^2.
// exp by scaling and squaring of a degree-16 Taylor polynomial
// (argument norm <= 1/2 after scaling: truncation below 1e-19).
// ---------------------------------------------------------------------------
__device__ void mat3_mul(const cplx* a, const cplx* b, cplx* o) {
    for (int x = 0; x < 3; ++x)
        for (int y = 0; y < 3; ++y) {
            cplx t = {0.0, 0.0};
            for (int q = 0; q < 3; ++q) {
                cplx m = cmul(a[3 * x + q], b[3 * q + y]);
                t.r += m.r; t.i += m.i;
            }
            o[3 * x + y] = t;
        }
}

__global__ void __launch_bounds__(256) k_md_update(double2* __restrict__ U, double2* __restrict__ P,
                                                   const double2* __restrict__ F, double dt_p,
                                                   double dt_u, int nlink, double* partial) {
    const int l = blockIdx.x * blockDim.x + threadIdx.x;
    double kin = 0;
    if (l < nlink) {
        cplx p[9];
        for (int q = 0; q < 9; ++q) p[q] = {P[(size_t)l * 9 + q].x, P[(size_t)l * 9 + q].y};
        if (F && dt_p != 0.0) {
            for (int q = 0; q < 9; ++q) {
                p[q].r -= dt_p * F[(size_t)l * 9 + q].x;
                p[q].i -= dt_p * F[(size_t)l * 9 + q].y;
            }
            for (int q = 0; q < 9; ++q) P[(size_t)l * 9 + q] = make_double2(p[q].r, p[q].i);
        }
        if (dt_u != 0.0) {
            cplx X[9];   // X = i dt_u P
            double nrm = 0;
            for (int q = 0; q < 9; ++q) {
                X[q] = {-dt_u * p[q].i, dt_u * p[q].r};
                nrm += X[q].r * X[q].r + X[q].i * X[q].i;
            }
            nrm = sqrt(nrm);
            int sq = 0;
            while (nrm > 0.5 && sq < 40) { nrm *= 0.5; ++sq; }
            const double scale = ldexp(1.0, -sq);
            for (int q = 0; q < 9; ++q) { X[q].r *= scale; X[q].i *= scale; }
            cplx E[9], T[9], W[9];
            for (int q = 0; q < 9; ++q) { E[q] = {q % 4 == 0 ? 1.0 : 0.0, 0.0}; T[q] = E[q]; }
            for (int nn = 1; nn <= 16; ++nn) {
                mat3_mul(T, X, W);
                const double inv = 1.0 / nn;
                for (int q = 0; q < 9; ++q) { T[q] = {W[q].r * inv, W[q].i * inv}; E[q].r += T[q].r; E[q].i += T[q].i; }
            }
            for (int r = 0; r < sq; ++r) {
                mat3_mul(E, E, W);
                for (int q = 0; q < 9; ++q) E[q] = W[q];
            }
            cplx u[9];
            for (int q = 0; q < 9; ++q) u[q] = {U[(size_t)l * 9 + q].x, U[(size_t)l * 9 + q].y};
            mat3_mul(E, u, W);
            for (int q = 0; q < 9; ++q) U[(size_t)l * 9 + q] = make_double2(W[q].r, W[q].i);
        }
        // tr(P^2) = sum_xy P_xy P_yx
        for (int x = 0; x < 3; ++x)
            for (int y = 0; y < 3; ++y) kin += cmul(p[3 * x + y], p[3 * y + x]).r;
    }
    if (partial) {
        __shared__ double red[4];
        double x = kin;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
        __syncthreads();
        if (threadIdx.x == 0) partial[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
    }
}

// The tile: extents of 4 along two directions and 2 along the other two, the
// pair that pads the lattice least.  Ties go to z and t: tiles are walked x
// first, so the workgroups of an XCD that run together cover x and y and
// share those faces in its L2, while the z and t faces, halved by the longer
// extents, come from beyond it (24^3x64, Ls = 24: 3.10 ms against 3.37 ms
// with the long extents along x and y).
//
// The split: one workgroup per tile walks its slice pairs in a row, 1.9 us each
// on an idle GPU, so up to 128 tiles (half of the 256 CUs) the pairs of a system
// are shared out to sqrt(Ls) workgroups (walks and the sum over them grow
// alike), at most two workgroups per CU.  A call at 4^4: Ls = 8 35.6 -> 29.5 us,
// Ls = 24 65.9 -> 33.9, Ls = 64 145 -> 41.7; 8^4, Ls = 24 69.4 -> 41.3 us;
// 8^3x16, Ls = 8 38.6 -> 37.6 us.  Beyond the line the second launch costs what
// the shorter walks save: 8^3x32 (256 tiles), Ls = 8 40.9 against 44.1 us, and
// below Ls = 8 too: 8^4, Ls = 4 29.0 against 32.2 us.
static ForceTile force_tiling(const int L[4], int Ls) {
    ForceTile ft{};
    for (int a = 0; a < 3; ++a)
        for (int b = a + 1; b < 4; ++b) {
            ForceTile c{};
            c.tiles = 1;
            for (int d = 0; d < 4; ++d) {
                c.lg[d] = d == a || d == b ? 2 : 1;
                c.n[d] = (L[d] + (1 << c.lg[d]) - 1) >> c.lg[d];
                c.tiles *= c.n[d];
            }
            if (ft.tiles == 0 || c.tiles <= ft.tiles) ft = c;
        }
    if (ft.tiles <= 128 && Ls >= 8) ft.split = std::min((int)std::sqrt((double)Ls), 256 / ft.tiles);
    return ft;
}

size_t force_workspace(const int L[4], int Ls) {
    const ForceTile ft = force_tiling(L, Ls);
    return (size_t)2 * ft.split * ft.tiles * 9 * 256 * sizeof(double2);
}

hipError_t launch_force(const void* U, const void* chiL, const void* chiR, double k, void* F, void* G,
                        const int L[4], int Ls, int aperiodic, void* part, hipStream_t st) {
    Geo g;
    for (int mu = 0; mu < 4; ++mu) g.L[mu] = L[mu];
    g.V = L[0] * L[1] * L[2] * L[3];
    g.Vh = g.V / 2;
    g.Ls = Ls;
    g.aperiodic = aperiodic;
    const ForceTile ft = force_tiling(L, Ls);
    const unsigned n = (unsigned)ft.tiles;
    if (ft.split == 0) {
        hipLaunchKernelGGL((k_force<false>), dim3(n), dim3(256), 0, st, (const double2*)chiL, (const double2*)chiR,
                           (const double2*)U, k, (double2*)F, (double2*)G, g, ft, (double2*)nullptr);
        return hipGetLastError();
    }
    if (!part) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_force<true>), dim3(n * 2 * ft.split), dim3(256), 0, st, (const double2*)chiL,
                       (const double2*)chiR, (const double2*)U, k, (double2*)F, (double2*)G, g, ft, (double2*)part);
    hipLaunchKernelGGL(k_force_finish, dim3(n), dim3(256), 0, st, (const double2*)part, (const double2*)U, k,
                       (double2*)F, (double2*)G, g, ft);
    return hipGetLastError();
}

int md_blocks(int nlink) { return (nlink + 255) / 256; }

// Scratch of the allocation-free MD update: the per-block partial sums of
// tr P^2 that k_md_update writes and k_reduce adds up.  Each GPU holds its
// own copy for the life of the process.  In host code the name below is not
// a device address: the host reaches the array only through the pointer
// md_scratch_address returns (hipGetSymbolAddress on the current device).
static __device__ __align__(256) double scratch[MD_SCRATCH_DOUBLES];

hipError_t md_scratch_address(double** out) {
    return hipGetSymbolAddress((void**)out, HIP_SYMBOL(scratch));
}

hipError_t launch_md_update(void* U, void* P, const void* F, double dt_p, double dt_u, int nlink,
                            double* partial, hipStream_t st) {
    hipLaunchKernelGGL(k_md_update, dim3(md_blocks(nlink)), dim3(256), 0, st, (double2*)U, (double2*)P,
                       (const double2*)F, dt_p, dt_u, nlink, partial);
    return hipGetLastError();
}

}  // namespace eofa
