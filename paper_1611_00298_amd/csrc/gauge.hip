// gauge.hip -- gauge action of the ensembles (Table 1: Iwasaki) and its force.
//
//   S_g = beta sum_x [ c0 sum_{mu<nu} (1 - Re tr W_1x1/3) + c1 sum_{mu!=nu} (1 - Re tr W_2x1/3) ]
// with c0 = 1 - 8 c1; W_2x1 is the loop two links long in mu and one in nu.
// c1 = -0.331 is the Iwasaki action, c1 = 0 the Wilson action.  Links are
// periodic in every direction (the fermion boundary phase is not part of U).
//
// Force: S_g depends on one link U_mu(x) through -(beta/3) Re tr(U_mu(x) Sigma)
// with Sigma the weighted sum of the staples (the rest of every loop through
// the link, walked from x+mu back to x).  With Omega = U Sigma and the
// convention of the fermion force (F = sum_a T^a d^a S, d^a along
// U -> exp(i eps T^a) U, T^a = lambda^a/2):
//   F = -(beta/12) (Y - tr(Y)/3),  Y = i (Omega - Omega^dag).
// Per plane (mu, nu), nu != mu, a link sits in two plaquettes and six
// rectangles: four long in mu (the link first or second along mu, nu up or
// down) and two long in nu (nu up or down).
//
// FP64 throughout, natural gauge layout U[mu][i][3][3] (i the natural site
// index); blocks are mapped to contiguous ranges per XCD so that neighbouring
// links are shared within one L2.
#include "internal.h"

namespace eofa {

namespace {

struct M3 {
    double2 e[9];
};

__device__ __forceinline__ M3 ldm(const double2* __restrict__ U, size_t link) {
    M3 m;
    const double2* p = U + link * 9;
#pragma unroll
    for (int q = 0; q < 9; ++q) m.e[q] = p[q];
    return m;
}

// a b
__device__ __forceinline__ M3 mul_nn(const M3& a, const M3& b) {
    M3 o;
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int y = 0; y < 3; ++y) {
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const double2 u = a.e[3 * x + q], v = b.e[3 * q + y];
                re = fma(u.x, v.x, fma(-u.y, v.y, re));
                im = fma(u.x, v.y, fma(u.y, v.x, im));
            }
            o.e[3 * x + y] = make_double2(re, im);
        }
    return o;
}
// a b^dag
__device__ __forceinline__ M3 mul_nd(const M3& a, const M3& b) {
    M3 o;
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int y = 0; y < 3; ++y) {
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) {   // a_xq conj(b_yq)
                const double2 u = a.e[3 * x + q], v = b.e[3 * y + q];
                re = fma(u.x, v.x, fma(u.y, v.y, re));
                im = fma(u.y, v.x, fma(-u.x, v.y, im));
            }
            o.e[3 * x + y] = make_double2(re, im);
        }
    return o;
}
// a^dag b
__device__ __forceinline__ M3 mul_dn(const M3& a, const M3& b) {
    M3 o;
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int y = 0; y < 3; ++y) {
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) {   // conj(a_qx) b_qy
                const double2 u = a.e[3 * q + x], v = b.e[3 * q + y];
                re = fma(u.x, v.x, fma(u.y, v.y, re));
                im = fma(u.x, v.y, fma(-u.y, v.x, im));
            }
            o.e[3 * x + y] = make_double2(re, im);
        }
    return o;
}
__device__ __forceinline__ M3 dag(const M3& a) {
    M3 o;
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int y = 0; y < 3; ++y) o.e[3 * x + y] = make_double2(a.e[3 * y + x].x, -a.e[3 * y + x].y);
    return o;
}
__device__ __forceinline__ M3 scaled(double s, const M3& a) {
    M3 o;
#pragma unroll
    for (int q = 0; q < 9; ++q) o.e[q] = make_double2(s * a.e[q].x, s * a.e[q].y);
    return o;
}
// o += s a
__device__ __forceinline__ void axpy(M3& o, double s, const M3& a) {
#pragma unroll
    for (int q = 0; q < 9; ++q) o.e[q] = make_double2(fma(s, a.e[q].x, o.e[q].x), fma(s, a.e[q].y, o.e[q].y));
}
// Re tr(a b^dag)
__device__ __forceinline__ double retr_nd(const M3& a, const M3& b) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < 9; ++q) t = fma(a.e[q].x, b.e[q].x, fma(a.e[q].y, b.e[q].y, t));
    return t;
}

// F = -(beta/12) (Y - tr Y / 3), Y = i (Omega - Omega^dag)
__device__ __forceinline__ M3 force_of(const M3& Om, double beta) {
    const double f = -beta / 12.0;
    const double trY = -2.0 * (Om.e[0].y + Om.e[4].y + Om.e[8].y);
    M3 o;
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int y = 0; y < 3; ++y) {
            const double2 a = Om.e[3 * x + y], b = Om.e[3 * y + x];
            // Y_xy = i (a - conj(b))
            double re = -(a.y + b.y), im = a.x - b.x;
            if (x == y) re -= trY / 3.0;
            o.e[3 * x + y] = make_double2(f * re, f * im);
        }
    return o;
}

struct Lat {
    int L[4];
    int stride[4];
    int V;
};

__device__ __forceinline__ void coords(const Lat& g, int i, int (&c)[4]) {
    int r = i;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        c[d] = r % g.L[d];
        r /= g.L[d];
    }
}

// natural index of x + a e_mu + b e_nu (periodic) for |a|, |b| <= 2 and
// every extent >= 2: one wrap per direction suffices
__device__ __forceinline__ int shift2(const Lat& g, const int (&c)[4], int i, int mu, int a, int nu, int b) {
    int cm = c[mu] + a, cn = c[nu] + b;
    cm = cm < 0 ? cm + g.L[mu] : (cm >= g.L[mu] ? cm - g.L[mu] : cm);
    cn = cn < 0 ? cn + g.L[nu] : (cn >= g.L[nu] ? cn - g.L[nu] : cn);
    return i + (cm - c[mu]) * g.stride[mu] + (cn - c[nu]) * g.stride[nu];
}

}  // namespace

// Force contributions of one plane, c1 != 0.  A workgroup takes a tile of at
// most 64 sites of a (mu, nu) plane and stages its U_mu and U_nu, two sites
// around it included, in LDS: every loop through a link lies in a plane, so
// this is all the plane's loops need (4.5 link reads per site and plane at
// 8x8, where one work-item per link reads 22 for each of the two links and is
// bound by the L2).  It then forms the corner products
//   P_mu(y) = U_mu(y) U_nu(y+mu),  P_nu(y) = U_nu(y) U_mu(y+nu)
// once for all loops that use them.  Wavefront (d, below) sums the loops above
// or below its lanes' links of direction d; with o the other direction,
// y = x - o, and the three-link detours
//   T(y) = P_o(y) U_o(y+d)^dag      for U_d(y), above     (at x+o)
//   D(y) = U_o(y-o)^dag P_d(y-o)    for U_d(y), below     (at x-o)
//   R(y) = P_d(y) U_d(y+o)^dag      for U_o(y), ahead
//   B(y) = U_d(y-d)^dag P_o(y-d)    for U_o(y), behind
// the staples are
//   above: U_o(x+d) [c0 P_o(x) + c1 (B(x) U_d(x+o) + U_o(x) T(x+o))]^dag + c1 R(x+d) P_o(x)^dag
//   below: [c0 P_d(y) + c1 (D(y) U_o(y+d) + U_d(y) R(y+d))]^dag U_o(y) + c1 P_d(y)^dag B(y)
// Per link and plane that is 16 products and its share of the corner products
// (22 without sharing).  Bound by FP64 arithmetic and LDS reads between
// barriers (47 and 39 % busy; LDS holds two workgroups per CU): the Iwasaki
// force at 24^3x64 takes 2.02 ms, the per-link form 3.73 ms.  Measured slower:
// workgroups that walk many tiles with the next tile's links in flight
// (2.2 ms), operands requested a product ahead (2.3 ms, spills), 8 wavefronts
// of half the chain each (2.8 ms, spills).
constexpr int GH = 2;           // staged sites around the tile
constexpr int GT_SITES = 64;    // most tile sites: a lane each
constexpr int GT_EXT = 152;     // most staged sites
constexpr int GT_MATS = 552;    // matrices in LDS: two workgroups per CU (8x8: 2 x 144 links, 2 x 132 corner products)

struct GPlane {
    int mu, nu;      // the plane
    int a, b;        // the other two directions
    int tm, tn;      // tile extents
    int nm, nn;      // tiles along mu and nu
    int nblk;        // workgroups of the plane
};

__global__ void __launch_bounds__(256, 2) k_gauge_force(const double2* __restrict__ U, double2* __restrict__ F, Lat g,
                                                        double beta, double c1, int accumulate, GPlane p0, GPlane p1) {
    constexpr int H = GH;
    constexpr int NU = (2 * GT_EXT * 9 + 255) / 256;     // words of links per work-item
    constexpr int NF = (2 * GT_SITES * 9 + 255) / 256;   // words of F per work-item
    extern __shared__ unsigned char smem_raw[];
    __shared__ int ext[GT_EXT];       // natural index of each staged site
    __shared__ int nat[GT_SITES];     // and of each tile site, -1: none
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int d = wave & 1;
    const bool below = wave >= 2;
    int blk = xcd_block(gridDim.x);
    const bool second = blk >= p0.nblk;
    const GPlane p = second ? p1 : p0;
    if (second) blk -= p0.nblk;
    const int i = lane % p.tm;
    int j = lane / p.tm;
    // 8x8: rows 0, 2, 1, 3, ..., so that the 16 lanes LDS serves together read different banks
    if (p.tm == 8 && p.tn == 8) j = (j & 4) | ((j & 1) << 1) | ((j >> 1) & 1);
    const int uw = p.tm + 2 * H, uh = p.tn + 2 * H, ne = uw * uh, np = uw * (uh - 1);
    {
        // planes next to each other along the first of the other two directions (x
        // where the plane does not hold it: neighbouring records share cache
        // lines), then the tiles of a plane
        const int base_a = (blk % g.L[p.a]) * g.stride[p.a];
        blk /= g.L[p.a];
        const int om = (blk % p.nm) * p.tm;
        blk /= p.nm;
        const int on = (blk % p.nn) * p.tn;
        blk /= p.nn;
        const int base = base_a + blk * g.stride[p.b];
        const int Lm = g.L[p.mu], Ln = g.L[p.nu];
        auto site = [&](int x, int y) {   // site (x, y) of the plane, any x, y >= -2
            return base + ((om + x + Lm) % Lm) * g.stride[p.mu] + ((on + y + Ln) % Ln) * g.stride[p.nu];
        };
        if (tid < ne) ext[tid] = site(tid % uw - H, tid / uw - H);
        if (tid < GT_SITES)
            nat[tid] = (j < p.tn && om + i < Lm && on + j < Ln) ? site(i, j) : -1;
    }
    __syncthreads();
    M3* Us = reinterpret_cast<M3*>(smem_raw);   // [2][uh][uw]
    M3* Ps = Us + 2 * ne;                       // [2][uh - 1][uw]
    {   // links: 9 consecutive work-items per record, all of a work-item's words in flight
        const d2v* Um = reinterpret_cast<const d2v*>(U + (size_t)p.mu * g.V * 9);
        const d2v* Un = reinterpret_cast<const d2v*>(U + (size_t)p.nu * g.V * 9);
        d2v* dst = reinterpret_cast<d2v*>(Us);
        const int n = 2 * ne * 9;
        d2v v[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int e = min(tid + 256 * u, n - 1), r = e / 9, c = e - 9 * r;
            v[u] = (r < ne ? Um : Un)[(size_t)ext[r < ne ? r : r - ne] * 9 + c];
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) dst[min(tid + 256 * u, n - 1)] = v[u];
    }
    __syncthreads();
    {   // P_mu at i >= 1, P_nu at j >= 1 (what the staples read), (i, j) counted from the staged corner
        const int wm = p.tm + 2 * (H - 1), hm = p.tn + H, wn = p.tm + H, n = wm * hm + wn * (p.tn + 2 * (H - 1));
        for (int e = tid; e < n; e += 256) {
            const int s = e >= wm * hm, q = s ? e - wm * hm : e, w = s ? wn : wm;
            const int k = (q / w + s) * uw + q % w + 1 - s;
            Ps[s * np + k] = mul_nn(Us[s * ne + k], Us[(1 - s) * ne + k + (s ? uw : 1)]);
        }
    }
    __syncthreads();
    // inactive lanes of a smaller tile repeat its first site
    const int li = j < p.tn ? i : 0, lj = j < p.tn ? j : 0;
    const int ud = d ? uw : 1, uo = d ? 1 : uw, k0 = (lj + H) * uw + li + H;
    const M3* Wd = Us + d * ne + k0;         // U_d, U_o, P_d, P_o at the link's site
    const M3* Wo = Us + (1 - d) * ne + k0;
    const M3* Qd = Ps + d * np + k0;
    const M3* Qo = Ps + (1 - d) * np + k0;
    const double c0 = 1.0 - 8.0 * c1;
    const M3* Vd = Wd - uo;   // the same at y = x - o
    const M3* Vo = Wo - uo;
    const M3* Rd = Qd - uo;
    const M3* Ro = Qo - uo;
    M3* X = Us + wave * 64 + lane;   // this work-item's slot once the staged links are read
    M3 S;
    if (!below) {
        M3 E = scaled(c0, Qo[0]);
        axpy(E, c1, mul_nn(mul_dn(Wd[-ud], Qo[-ud]), Wd[uo]));
        axpy(E, c1, mul_nn(Wo[0], mul_nd(Qo[uo], Wo[uo + ud])));
        S = mul_nd(Wo[ud], E);
        axpy(S, c1, mul_nd(mul_nd(Qd[ud], Wd[ud + uo]), Qo[0]));
    } else {
        M3 E = scaled(c0, Rd[0]);
        axpy(E, c1, mul_nn(mul_dn(Vo[-uo], Rd[-uo]), Vo[ud]));
        axpy(E, c1, mul_nn(Vd[0], mul_nd(Rd[ud], Vd[ud + uo])));
        S = mul_dn(E, Vo[0]);
        axpy(S, c1, mul_dn(Rd[0], mul_dn(Vd[-ud], Ro[-ud])));
    }
    S = mul_nn(Wd[0], S);
    __syncthreads();   // the staged links are read: their space takes the results
    if (below) X[0] = S;
    __syncthreads();
    // Omega = U Sigma of both halves
    if (!below) {
        axpy(S, 1.0, X[128]);
        X[0] = force_of(S, beta);   // slots 0..127: direction d, tile site
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NF; ++u) {
        const int e = tid + 256 * u, r = e / 9, c = e - 9 * r;
        if (e >= 2 * GT_SITES * 9) break;
        const int s = nat[r & (GT_SITES - 1)];
        if (s < 0) continue;
        d2v x = reinterpret_cast<const d2v*>(Us)[e];
        d2v* q = reinterpret_cast<d2v*>(F) + ((size_t)(r < GT_SITES ? p.mu : p.nu) * g.V + s) * 9 + c;
        if (accumulate) x += *q;
        *q = x;
    }
}

// The plaquette part alone (c1 = 0): one work-item per link l = mu V + i.  Its
// 25 link reads and 13 products leave too little to share: at 24^3x64 it takes
// 0.95 ms, the plane tiles 1.5 ms (three passes over F).  The nine loads of a
// link touch the same lines, which have to last in the 32 KB L1 from the first
// to the last: one wavefront per SIMD, and as few links requested at a time as
// a product needs (1.05 ms without the scheduling barriers, 1.35 ms with two
// wavefronts per SIMD, 2.3 ms with three).
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) k_wilson_force(const double2* __restrict__ U, double2* __restrict__ F,
                                                      Lat g, double beta, int accumulate) {
    const int l = xcd_block(gridDim.x) * blockDim.x + threadIdx.x;
    if (l >= 4 * g.V) return;
    const int mu = l / g.V, i = l - mu * g.V;
    int c[4];
    coords(g, i, c);
    const size_t V = (size_t)g.V;
    auto lk = [&](int d, int site) { return ldm(U, (size_t)d * V + site); };
    M3 sig;
#pragma unroll
    for (int q = 0; q < 9; ++q) sig.e[q] = make_double2(0.0, 0.0);
#pragma unroll 1
    for (int nu = 0; nu < 4; ++nu) {
        if (nu == mu) continue;
        auto at = [&](int a, int b) { return shift2(g, c, i, mu, a, nu, b); };
        // U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
        const M3 B = mul_nd(lk(nu, at(1, 0)), lk(mu, at(0, 1)));
        __builtin_amdgcn_sched_barrier(0);   // fewer links' lines in use at a time
        axpy(sig, 1.0, mul_nd(B, lk(nu, i)));
        __builtin_amdgcn_sched_barrier(0);
        // U_nu(x+mu-nu)^dag U_mu(x-nu)^dag U_nu(x-nu)
        const M3 D = dag(mul_nn(lk(mu, at(0, -1)), lk(nu, at(1, -1))));
        __builtin_amdgcn_sched_barrier(0);
        axpy(sig, 1.0, mul_nn(D, lk(nu, at(0, -1))));
    }
    const M3 Om = mul_nn(lk(mu, i), sig);
    const M3 o = force_of(Om, beta);
    double2* Fl = F + (size_t)l * 9;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        double2 v = o.e[q];
        if (accumulate) {
            v.x += Fl[q].x;
            v.y += Fl[q].y;
        }
        Fl[q] = v;
    }
}

// One work-item per site: c0 sum_{mu<nu} (1 - Re tr W_1x1/3) + c1 sum_{mu!=nu} (1 - Re tr W_2x1/3),
// summed per workgroup into partial[block].
__global__ void __launch_bounds__(256) k_gauge_action(const double2* __restrict__ U, Lat g, double c1,
                                                      double* __restrict__ partial) {
    const int i = xcd_block(gridDim.x) * blockDim.x + threadIdx.x;
    double acc = 0.0;
    if (i < g.V) {
        const double c0 = 1.0 - 8.0 * c1;
        const bool rect = c1 != 0.0;
        int c[4];
        coords(g, i, c);
        const size_t V = (size_t)g.V;
        auto lk = [&](int d, int site) { return ldm(U, (size_t)d * V + site); };
#pragma unroll 1
        for (int mu = 0; mu < 4; ++mu) {
#pragma unroll 1
            for (int nu = 0; nu < 4; ++nu) {
                if (nu == mu) continue;
                auto at = [&](int a, int b) { return shift2(g, c, i, mu, a, nu, b); };
                const M3 um = lk(mu, i), un = lk(nu, i);
                if (mu < nu) {   // U_mu(x) U_nu(x+mu) [U_nu(x) U_mu(x+nu)]^dag
                    const double p = retr_nd(mul_nn(um, lk(nu, at(1, 0))), mul_nn(un, lk(mu, at(0, 1))));
                    acc = fma(c0, 1.0 - p / 3.0, acc);
                }
                if (rect) {      // U_mu(x) U_mu(x+mu) U_nu(x+2mu) [U_nu(x) U_mu(x+nu) U_mu(x+mu+nu)]^dag
                    const M3 a = mul_nn(mul_nn(um, lk(mu, at(1, 0))), lk(nu, at(2, 0)));
                    const M3 b = mul_nn(mul_nn(un, lk(mu, at(0, 1))), lk(mu, at(1, 1)));
                    acc = fma(c1, 1.0 - retr_nd(a, b) / 3.0, acc);
                }
            }
        }
    }
    __shared__ double red[4];
    double x = acc;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

static Lat make_lat(const int L[4]) {
    Lat g;
    int s = 1;
    for (int d = 0; d < 4; ++d) {
        g.L[d] = L[d];
        g.stride[d] = s;
        s *= L[d];
    }
    g.V = s;
    return g;
}

int gauge_action_blocks(int V) { return (V + 255) / 256; }

// Tiles of one plane: the fewest tiles of at most GT_SITES sites whose links
// and corner products fit GT_MATS matrices (8x8 where it divides; 10x6, 7x9
// and the like for uneven extents), the squarest of those.
static GPlane make_plane(const int L[4], int mu, int nu) {
    GPlane p{};
    p.mu = mu;
    p.nu = nu;
    int other[2], k = 0;
    for (int d = 0; d < 4; ++d)
        if (d != mu && d != nu) other[k++] = d;
    p.a = other[0];
    p.b = other[1];
    long best = -1;
    for (int nm = 1; nm <= L[mu] && (best < 0 || nm <= best >> 20); ++nm)
        for (int nn = 1; nn <= L[nu]; ++nn) {
            const int tm = (L[mu] + nm - 1) / nm, tn = (L[nu] + nn - 1) / nn;
            const int uw = tm + 2 * GH, uh = tn + 2 * GH;
            if (tm * tn > GT_SITES || uw * uh > GT_EXT || 2 * uw * uh + 2 * uw * (uh - 1) > GT_MATS) continue;
            const long score = ((long)nm * nn << 20) + (tm > tn ? tm - tn : tn - tm);
            if (best < 0 || score < best) {
                best = score;
                p.nm = nm;
                p.nn = nn;
                p.tm = tm;
                p.tn = tn;
            }
            break;   // more tiles along nu only raise the count
        }
    p.nblk = p.nm * p.nn * L[p.a] * L[p.b];
    return p;
}

// The six planes in three launches of two planes without a common direction,
// so that every launch adds one plane's contribution to every link.
hipError_t launch_gauge_force(const void* U, void* F, const int L[4], double beta, double c1, int accumulate,
                              hipStream_t st) {
    const Lat g = make_lat(L);
    if (c1 == 0.0) {
        hipLaunchKernelGGL(k_wilson_force, dim3((4 * g.V + 255) / 256), dim3(256), 0, st, (const double2*)U,
                           (double2*)F, g, beta, accumulate);
        return hipGetLastError();
    }
    const int pairs[3][4] = {{0, 1, 2, 3}, {0, 2, 1, 3}, {0, 3, 1, 2}};
    for (int k = 0; k < 3; ++k) {
        const GPlane p0 = make_plane(L, pairs[k][0], pairs[k][1]), p1 = make_plane(L, pairs[k][2], pairs[k][3]);
        hipLaunchKernelGGL(k_gauge_force, dim3((unsigned)(p0.nblk + p1.nblk)), dim3(256), GT_MATS * sizeof(M3), st,
                           (const double2*)U, (double2*)F, g, beta, c1, accumulate || k > 0, p0, p1);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_gauge_action(const void* U, const int L[4], double c1, double* partial, hipStream_t st) {
    const Lat g = make_lat(L);
    hipLaunchKernelGGL(k_gauge_action, dim3(gauge_action_blocks(g.V)), dim3(256), 0, st, (const double2*)U, g, c1,
                       partial);
    return hipGetLastError();
}

}  // namespace eofa
