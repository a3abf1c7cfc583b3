// Differentiable Monte Carlo (Methods, Algorithm 2) for the Ising model on
// gfx950: the relaxed checkerboard chain on continuous spins with one coupling
// per bond, and its reverse-mode gradient by replaying the chain backwards.
//
// One colour pass (colour c = (x + y) & 1, pass p = 2t + c) updates every
// site of colour c from the current spins:
//     hloc = Jx[y][x] s(y,x+1) + Jx[y][x-1] s(y,x-1) + Jy[y][x] s(y+1,x)
//            + Jy[y-1][x] s(y-1,x) + h
//     P = exp(min(-2 beta s hloc, 80)),  q = 1 / (1 + exp(-alpha (P - r))),
//     s <- s (1 - 2 q)          (the flip s' = -s mixed in with weight q)
// with r = (word >> 8) 2^-24 from Philox4x32-10 counter (k >> 2, p, rid, 3),
// word k & 3, k = y Lx/2 + (x >> 1).  A lane handles the four sites of one
// Philox block.  Spins and couplings are FP32, row-major [R][Ly][Lx].
//
// Backward of a pass, with a = dL/ds_new at a colour-c site and
// w = 4 alpha beta q (1 - q) P:
//     dL/ds_old = a ((1 - 2q) + w s_old hloc)
//     t = a w s_old^2  = dL/dhloc
//     dL/dJ(bond to n) += t s_n,   dL/ds_n += t J(bond to n)   (n of colour 1-c)
// Every bond has exactly one colour-c end, so the coupling gradients of a
// pass are written by one lane each.  The neighbour terms t J go to sites of
// the other colour, whose adjoints are only read again by the next pass of
// the replay: that pass adds them while it loads its own adjoint (the t of
// the previous pass is kept in a second plane of the work buffer), and one
// gather kernel adds those of the last pass.  The pre-pass spins of colour c
// are saved by the forward pass (one colour plane per pass), which is what
// the backward replay restores.
//
// Two layouts of the lane work: when Lx is a multiple of 8 (and every buffer
// is 16-byte aligned) the four sites of a Philox block are one 8-float span
// of a row, and a lane loads the spans of rows y-1, y, y+1 and of the
// couplings with 16-byte loads; otherwise every site is addressed on its own.
#include "dmc_internal.hpp"

namespace spinmc {

namespace {

constexpr uint32_t kTagDmc = 3u;

__device__ __forceinline__ int wrapd(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

struct DmcSite {
    int y, x;
    size_t i;  // natural index within the replica
};

__device__ __forceinline__ DmcSite dmc_site(int k, int W, int c) {
    DmcSite d;
    d.y = k / W;
    d.x = 2 * (k - d.y * W) + ((d.y + c) & 1);
    d.i = (size_t)d.y * (2 * W) + d.x;
    return d;
}

// the update of one site from its neighbourhood: local field, P and q
struct DmcUpd {
    float hloc, P, q;
};

__device__ __forceinline__ DmcUpd dmc_update(float sv, float jr, float sr, float jl, float sl,
                                             float jd, float sd, float ju, float su, float beta,
                                             float alpha, float h, uint32_t word) {
    DmcUpd U;
    U.hloc = jr * sr + jl * sl + jd * sd + ju * su + h;
    // exponent capped at 80: beyond it q is exactly 1 anyway, and an infinite
    // P would turn the backward's q (1 - q) P into 0 * inf
    U.P = expf(fminf(-beta * (2.0f * sv * U.hloc), 80.0f));
    const float r = (float)(word >> 8) * 0x1p-24f;
    U.q = 1.0f / (1.0f + expf(-alpha * (U.P - r)));
    return U;
}

// neighbourhood of a site addressed on its own
struct DmcNb {
    float sr, sl, sd, su;  // neighbour spins
    float jr, jl, jd, ju;  // couplings of the four bonds
    int xr, xl, yd, yu;
};

__device__ __forceinline__ DmcNb dmc_nb(const float* s, const float* Jx, const float* Jy, int Lx,
                                        int Ly, int y, int x) {
    DmcNb N;
    N.xr = wrapd(x + 1, Lx);
    N.xl = wrapd(x - 1, Lx);
    N.yd = wrapd(y + 1, Ly);
    N.yu = wrapd(y - 1, Ly);
    const size_t row = (size_t)y * Lx;
    N.sr = s[row + N.xr];
    N.sl = s[row + N.xl];
    N.sd = s[(size_t)N.yd * Lx + x];
    N.su = s[(size_t)N.yu * Lx + x];
    N.jr = Jx[row + x];
    N.jl = Jx[row + N.xl];
    N.jd = Jy[row + x];
    N.ju = Jy[(size_t)N.yu * Lx + x];
    return N;
}

// An 8-float span of a row held as two float4 values (registers only: the
// sites are picked by value selects, never by an index into a local array).
struct Row8 {
    float4 a, b;
};

__device__ __forceinline__ Row8 ld8(const float* p) {
    return Row8{*reinterpret_cast<const float4*>(p), *reinterpret_cast<const float4*>(p + 4)};
}

__device__ __forceinline__ float el4(const float4& v, int i) {
    return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w));
}

// element i (0..7, a compile-time constant after unrolling) of a span
__device__ __forceinline__ float el8(const Row8& r, int i) { return i < 4 ? el4(r.a, i) : el4(r.b, i - 4); }

// element i of the span extended by one column on each side: index 0 is the
// column left of the span, 9 the one right of it (both are e: a lane needs
// only the side its parity reaches)
__device__ __forceinline__ float el10(const Row8& r, float e, int i) {
    return (i == 0 || i == 9) ? e : el8(r, i - 1);
}

// the same for a span extended on the left only (index 0)
__device__ __forceinline__ float el9(const Row8& r, float e, int i) {
    return i == 0 ? e : el8(r, i - 1);
}

__device__ __forceinline__ float pick(bool o, float odd, float even) { return o ? odd : even; }

// the span r with the four own sites (odd offsets if o, even otherwise)
// replaced by v, written as two 16-byte stores
__device__ __forceinline__ void store_span(float* p, const Row8& r, bool o, const float* v) {
    float4 A = r.a, B = r.b;
    if (o) {
        A.y = v[0]; A.w = v[1]; B.y = v[2]; B.w = v[3];
    } else {
        A.x = v[0]; A.z = v[1]; B.x = v[2]; B.z = v[3];
    }
    *reinterpret_cast<float4*>(p) = A;
    *reinterpret_cast<float4*>(p + 4) = B;
}

// Span of one Philox block when Lx % 8 == 0: block b covers row y, columns
// x0 .. x0 + 7 with x0 = 8 (b mod Lx/8); its sites are x0 + 2u + par,
// par = (y + c) & 1.  xe is the column beyond the span that the sites'
// horizontal neighbours reach (x0 - 1 for par 0, x0 + 8 for par 1), xj the
// bond left of the span (x0 - 1).
struct Span8 {
    int y, x0, par, yd, yu, xe, xj;
};

__device__ __forceinline__ Span8 span8(int b, int Lx, int Ly, int c) {
    Span8 S;
    const int G = Lx >> 3;
    S.y = b / G;
    S.x0 = 8 * (b - S.y * G);
    S.par = (S.y + c) & 1;
    S.yd = S.y + 1 == Ly ? 0 : S.y + 1;
    S.yu = S.y == 0 ? Ly - 1 : S.y - 1;
    S.xj = S.x0 == 0 ? Lx - 1 : S.x0 - 1;
    S.xe = S.par ? (S.x0 + 8 == Lx ? 0 : S.x0 + 8) : S.xj;
    return S;
}

}  // namespace

// ---- forward ---------------------------------------------------------------

__global__ void __launch_bounds__(256) k_dmc_pass(DmcArgs a, int c, uint32_t p, float* save) {
    const int W = a.Lx >> 1;
    const int n_sites = a.Ly * W;
    const int n_blocks = (n_sites + 3) >> 2;
    const int r = blockIdx.y;
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_blocks) return;
    const size_t off = (size_t)r * a.Lx * a.Ly;
    float* s = a.s + off;
    const float* Jx = a.Jx + off;
    const float* Jy = a.Jy + off;
    float* sv_save = save + (size_t)r * n_sites;
    uint32_t w[4];
    philox4x32_10((uint32_t)b, p, a.rid0 + (uint32_t)r, kTagDmc, a.key0, a.key1, w);
    // every load of the four sites first, then the stores (the buffers may
    // alias as far as the compiler knows); no two of a lane's sites share a
    // bond, since every bond has one end of each colour
    float snew[4], sold[4];
    size_t idx[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int k = 4 * b + u;
        idx[u] = 0;
        snew[u] = sold[u] = 0.f;
        if (k >= n_sites) continue;
        const DmcSite d = dmc_site(k, W, c);
        idx[u] = d.i;
        const float sv = s[d.i];
        const DmcNb N = dmc_nb(s, Jx, Jy, a.Lx, a.Ly, d.y, d.x);
        const DmcUpd U = dmc_update(sv, N.jr, N.sr, N.jl, N.sl, N.jd, N.sd, N.ju, N.su, a.beta,
                                    a.alpha, a.h, w[u]);
        sold[u] = sv;
        snew[u] = sv * (1.0f - 2.0f * U.q);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (4 * b + u < n_sites) {
            sv_save[4 * b + u] = sold[u];
            s[idx[u]] = snew[u];
        }
}

// Lx % 8 == 0: rows y-1, y, y+1 of the spins and the coupling rows as 8-float
// spans; the own sites and their neighbours are picked by par.
// Offsets within a replica are 32-bit (Lx Ly <= 2^28), on a replica base that
// is uniform over the workgroup.
__device__ __forceinline__ void pass8_block(const DmcArgs& a, int c, uint32_t p, float* save,
                                            int r, int b, int n_blocks) {
    const int Lx = a.Lx;
    const Span8 P8 = span8(b, Lx, a.Ly, c);
    const size_t off = (size_t)r * Lx * a.Ly;
    float* s = a.s + off;
    const float* Jx = a.Jx + off;
    const float* Jy = a.Jy + off;
    const uint32_t rw = (uint32_t)P8.y * Lx, ro = rw + P8.x0, rd = (uint32_t)P8.yd * Lx + P8.x0,
                   ru = (uint32_t)P8.yu * Lx + P8.x0;
    // S: spins of row y over the span (plus the column beyond it that par
    // reaches), X: Jx of row y (plus the bond left of the span)
    const Row8 S = ld8(s + ro), D = ld8(s + rd), U = ld8(s + ru);
    const float se = s[rw + P8.xe];
    const Row8 X = ld8(Jx + ro), Y0 = ld8(Jy + ro), Y1 = ld8(Jy + ru);
    const float xe = Jx[rw + P8.xj];
    uint32_t w[4];
    philox4x32_10((uint32_t)b, p, a.rid0 + (uint32_t)r, kTagDmc, a.key0, a.key1, w);
    const bool o = P8.par != 0;
    float sold[4], snew[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const float sv = pick(o, el10(S, se, 2 * u + 2), el10(S, se, 2 * u + 1));
        const float sl = pick(o, el10(S, se, 2 * u + 1), el10(S, se, 2 * u));
        const float sr = pick(o, el10(S, se, 2 * u + 3), el10(S, se, 2 * u + 2));
        const float jr = pick(o, el9(X, xe, 2 * u + 2), el9(X, xe, 2 * u + 1));
        const float jl = pick(o, el9(X, xe, 2 * u + 1), el9(X, xe, 2 * u));
        const float sd = pick(o, el8(D, 2 * u + 1), el8(D, 2 * u));
        const float su = pick(o, el8(U, 2 * u + 1), el8(U, 2 * u));
        const float jd = pick(o, el8(Y0, 2 * u + 1), el8(Y0, 2 * u));
        const float ju = pick(o, el8(Y1, 2 * u + 1), el8(Y1, 2 * u));
        const DmcUpd Q = dmc_update(sv, jr, sr, jl, sl, jd, sd, ju, su, a.beta, a.alpha, a.h, w[u]);
        sold[u] = sv;
        snew[u] = sv * (1.0f - 2.0f * Q.q);
    }
    *reinterpret_cast<float4*>(save + (size_t)r * (4 * n_blocks) + 4 * (uint32_t)b) =
        make_float4(sold[0], sold[1], sold[2], sold[3]);
    // the whole span is written back, the other colour's values unchanged:
    // full cache lines instead of every other word (partial lines cost HBM
    // time), and no other lane writes the span during the pass
    store_span(s + ro, S, o, snew);
}

__global__ void __launch_bounds__(256) k_dmc_pass8(DmcArgs a, int c, uint32_t p, float* save) {
    const int n_blocks = a.Ly * (a.Lx >> 3);
    const int b = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (b >= n_blocks) return;
    pass8_block(a, c, p, save, blockIdx.y, b, n_blocks);
}

// ---- backward --------------------------------------------------------------

// tin: t of the pass replayed before this one (sites of colour 1 - c, the
// neighbours), or null for the first replayed pass; tout: t of this pass.
__global__ void __launch_bounds__(256) k_dmc_back(DmcArgs a, int c, uint32_t p,
                                                  const float* save, float* gs, float* gJx,
                                                  float* gJy, const float* tin, float* tout) {
    const int W = a.Lx >> 1;
    const int n_sites = a.Ly * W;
    const int n_blocks = (n_sites + 3) >> 2;
    const int r = blockIdx.y;
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_blocks) return;
    const size_t off = (size_t)r * a.Lx * a.Ly;
    float* s = a.s + off;
    const float* Jx = a.Jx + off;
    const float* Jy = a.Jy + off;
    float* g = gs + off;
    float* gx = gJx + off;
    float* gy = gJy + off;
    const float* sv_save = save + (size_t)r * n_sites;
    const float* ti = tin ? tin + (size_t)r * n_sites : nullptr;
    float* to = tout + (size_t)r * n_sites;
    uint32_t w[4];
    philox4x32_10((uint32_t)b, p, a.rid0 + (uint32_t)r, kTagDmc, a.key0, a.key1, w);
    // phase 1: every load of the four sites (including the coupling
    // gradients they add to); phase 2: every store
    float gout[4], tv[4], sold[4], gr[4], gl[4], gd[4], gu[4];
    size_t ii[4], ir[4], il[4], iu[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int k = 4 * b + u;
        gout[u] = tv[u] = sold[u] = gr[u] = gl[u] = gd[u] = gu[u] = 0.f;
        ii[u] = ir[u] = il[u] = iu[u] = 0;
        if (k >= n_sites) continue;
        const DmcSite d = dmc_site(k, W, c);
        const float sv = sv_save[k];
        const DmcNb N = dmc_nb(s, Jx, Jy, a.Lx, a.Ly, d.y, d.x);
        const DmcUpd U = dmc_update(sv, N.jr, N.sr, N.jl, N.sl, N.jd, N.sd, N.ju, N.su, a.beta,
                                    a.alpha, a.h, w[u]);
        float av = g[d.i];
        if (ti)  // within-colour index of (y', x'): y' W + (x' >> 1)
            av += N.jr * ti[d.y * W + (N.xr >> 1)] + N.jl * ti[d.y * W + (N.xl >> 1)] +
                  N.jd * ti[N.yd * W + (d.x >> 1)] + N.ju * ti[N.yu * W + (d.x >> 1)];
        const float wq = 4.0f * a.alpha * a.beta * U.q * (1.0f - U.q) * U.P;
        gout[u] = av * ((1.0f - 2.0f * U.q) + wq * sv * U.hloc);
        const float t = av * wq * sv * sv;
        tv[u] = t;
        sold[u] = sv;
        const size_t row = (size_t)d.y * a.Lx;
        ii[u] = d.i;
        ir[u] = row + d.x;
        il[u] = row + N.xl;
        iu[u] = (size_t)N.yu * a.Lx + d.x;
        gr[u] = gx[ir[u]] + t * N.sr;
        gl[u] = gx[il[u]] + t * N.sl;
        gd[u] = gy[ir[u]] + t * N.sd;
        gu[u] = gy[iu[u]] + t * N.su;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int k = 4 * b + u;
        if (k >= n_sites) continue;
        g[ii[u]] = gout[u];
        to[k] = tv[u];
        gx[ir[u]] = gr[u];
        gx[il[u]] = gl[u];
        gy[ir[u]] = gd[u];
        gy[iu[u]] = gu[u];
        s[ii[u]] = sold[u];  // the state before this pass
    }
}

// Lx % 8 == 0: the spans of the spins, couplings, adjoints and coupling
// gradients of rows y-1, y, y+1 as 16-byte loads.
__device__ __forceinline__ void back8_block(const DmcArgs& a, int c, uint32_t p,
                                            const float* save, float* gs, float* gJx, float* gJy,
                                            const float* tin, float* tout, int r, int b,
                                            int n_blocks) {
    const int Lx = a.Lx;
    const int W = Lx >> 1;
    const int n_sites = 4 * n_blocks;
    const Span8 P8 = span8(b, Lx, a.Ly, c);
    const size_t off = (size_t)r * Lx * a.Ly;
    float* s = a.s + off;
    const float* Jx = a.Jx + off;
    const float* Jy = a.Jy + off;
    float* g = gs + off;
    float* gx = gJx + off;
    float* gy = gJy + off;
    const uint32_t rw = (uint32_t)P8.y * Lx, ro = rw + P8.x0, rd = (uint32_t)P8.yd * Lx + P8.x0,
                   ru = (uint32_t)P8.yu * Lx + P8.x0;
    // as in the forward; G: adjoints of row y, GX: Jx gradients of row y
    // (plus the bond left of the span), GY0 / GY1: Jy gradients of rows y and
    // y - 1; T: t of the colour 1 - c sites of row y over the span (plus the
    // one beyond it that par reaches), TD / TU: the same in rows y + 1, y - 1
    const float4 sold4 = *reinterpret_cast<const float4*>(save + (size_t)r * n_sites +
                                                          4 * (uint32_t)b);
    const float sold[4] = {sold4.x, sold4.y, sold4.z, sold4.w};
    const Row8 S = ld8(s + ro), D = ld8(s + rd), U = ld8(s + ru);
    const float se = s[rw + P8.xe];
    const Row8 X = ld8(Jx + ro), Y0 = ld8(Jy + ro), Y1 = ld8(Jy + ru);
    const float xe = Jx[rw + P8.xj];
    const Row8 G = ld8(g + ro), GX = ld8(gx + ro), GY0 = ld8(gy + ro), GY1 = ld8(gy + ru);
    const float gxe = gx[rw + P8.xj];
    float4 T = make_float4(0.f, 0.f, 0.f, 0.f), TD = T, TU = T;
    float te = 0.f;
    if (tin) {
        // within-colour indices y' W + x0 / 2 + u (16-byte aligned)
        const float* ti = tin + (size_t)r * n_sites;
        T = *reinterpret_cast<const float4*>(ti + 4 * (uint32_t)b);
        te = ti[(uint32_t)P8.y * W + (P8.xe >> 1)];
        TD = *reinterpret_cast<const float4*>(ti + (uint32_t)P8.yd * W + (P8.x0 >> 1));
        TU = *reinterpret_cast<const float4*>(ti + (uint32_t)P8.yu * W + (P8.x0 >> 1));
    }
    uint32_t w[4];
    philox4x32_10((uint32_t)b, p, a.rid0 + (uint32_t)r, kTagDmc, a.key0, a.key1, w);
    const bool o = P8.par != 0;
    float gout[4], tv[4], gxl[4], gxr[4], gyd[4], gyu[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const float sv = sold[u];
        const float sl = pick(o, el10(S, se, 2 * u + 1), el10(S, se, 2 * u));
        const float sr = pick(o, el10(S, se, 2 * u + 3), el10(S, se, 2 * u + 2));
        const float jr = pick(o, el9(X, xe, 2 * u + 2), el9(X, xe, 2 * u + 1));
        const float jl = pick(o, el9(X, xe, 2 * u + 1), el9(X, xe, 2 * u));
        const float sd = pick(o, el8(D, 2 * u + 1), el8(D, 2 * u));
        const float su = pick(o, el8(U, 2 * u + 1), el8(U, 2 * u));
        const float jd = pick(o, el8(Y0, 2 * u + 1), el8(Y0, 2 * u));
        const float ju = pick(o, el8(Y1, 2 * u + 1), el8(Y1, 2 * u));
        const DmcUpd Q = dmc_update(sv, jr, sr, jl, sl, jd, sd, ju, su, a.beta, a.alpha, a.h, w[u]);
        float av = pick(o, el8(G, 2 * u + 1), el8(G, 2 * u));
        if (tin) {
            // T extended: index 0 = te (left, par 0), 1..4 = T, 5 = te (right, par 1)
            const float tl = pick(o, el4(T, u), u == 0 ? te : el4(T, u - 1));
            const float tr = pick(o, u == 3 ? te : el4(T, u + 1), el4(T, u));
            av += jr * tr + jl * tl + jd * el4(TD, u) + ju * el4(TU, u);
        }
        const float wq = 4.0f * a.alpha * a.beta * Q.q * (1.0f - Q.q) * Q.P;
        gout[u] = av * ((1.0f - 2.0f * Q.q) + wq * sv * Q.hloc);
        const float t = av * wq * sv * sv;
        tv[u] = t;
        gxr[u] = pick(o, el9(GX, gxe, 2 * u + 2), el9(GX, gxe, 2 * u + 1)) + t * sr;
        gxl[u] = pick(o, el9(GX, gxe, 2 * u + 1), el9(GX, gxe, 2 * u)) + t * sl;
        gyd[u] = pick(o, el8(GY0, 2 * u + 1), el8(GY0, 2 * u)) + t * sd;
        gyu[u] = pick(o, el8(GY1, 2 * u + 1), el8(GY1, 2 * u)) + t * su;
    }
    *reinterpret_cast<float4*>(tout + (size_t)r * n_sites + 4 * (uint32_t)b) =
        make_float4(tv[0], tv[1], tv[2], tv[3]);
    // the horizontal bonds of the span's sites: columns x0 .. x0 + 7 for
    // par 1; x0 - 1 .. x0 + 6 for par 0 (x0 + 7 belongs to the next span)
    if (o) {
        *reinterpret_cast<float4*>(gx + ro) = make_float4(gxl[0], gxr[0], gxl[1], gxr[1]);
        *reinterpret_cast<float4*>(gx + ro + 4) = make_float4(gxl[2], gxr[2], gxl[3], gxr[3]);
    } else {
        gx[rw + P8.xj] = gxl[0];
        *reinterpret_cast<float4*>(gx + ro) = make_float4(gxr[0], gxl[1], gxr[1], gxl[2]);
        gx[ro + 4] = gxr[2];
        gx[ro + 5] = gxl[3];
        gx[ro + 6] = gxr[3];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t x = 2 * u + P8.par;
        gy[ro + x] = gyd[u];
        gy[ru + x] = gyu[u];
    }
    // whole spans, as in the forward: the adjoints and the state before
    // this pass at the own sites, the other colour's values unchanged
    store_span(g + ro, G, o, gout);
    store_span(s + ro, S, o, sold);
}

__global__ void __launch_bounds__(256) k_dmc_back8(DmcArgs a, int c, uint32_t p,
                                                   const float* save, float* gs, float* gJx,
                                                   float* gJy, const float* tin, float* tout) {
    const int n_blocks = a.Ly * (a.Lx >> 3);
    const int b = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (b >= n_blocks) return;
    back8_block(a, c, p, save, gs, gJx, gJy, tin, tout, blockIdx.y, b, n_blocks);
}

// dL/ds_n += sum over the four colour-c neighbours i of t_i J(i, n), for the
// sites n of colour 1 - c.
__global__ void __launch_bounds__(256) k_dmc_gather(DmcArgs a, int c, float* gs,
                                                    const float* work) {
    const int W = a.Lx >> 1;
    const int n_sites = a.Ly * W;
    const int r = blockIdx.y;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n_sites) return;
    const size_t off = (size_t)r * a.Lx * a.Ly;
    const float* Jx = a.Jx + off;
    const float* Jy = a.Jy + off;
    const float* tw = work + (size_t)r * n_sites;
    const DmcSite d = dmc_site(k, W, 1 - c);
    const int Lx = a.Lx, Ly = a.Ly;
    const int xr = wrapd(d.x + 1, Lx), xl = wrapd(d.x - 1, Lx);
    const int yd = wrapd(d.y + 1, Ly), yu = wrapd(d.y - 1, Ly);
    const float tr = tw[d.y * W + (xr >> 1)], tl = tw[d.y * W + (xl >> 1)];
    const float td = tw[yd * W + (d.x >> 1)], tu = tw[yu * W + (d.x >> 1)];
    const size_t row = (size_t)d.y * Lx;
    const float acc = Jx[row + d.x] * tr + Jx[row + xl] * tl + Jy[row + d.x] * td +
                      Jy[(size_t)yu * Lx + d.x] * tu;
    gs[off + d.i] += acc;
}

// ---- resident chain ----------------------------------------------------------
// All passes of a call in one launch, one workgroup per replica.  A lane owns
// NI consecutive rows (NI even, from a row that NI divides, so that every
// row's parity is known at compile time) of an 8-column span for the whole
// launch and keeps their couplings in registers -- eight bonds and the one
// left of the span per row, the vertical bonds of its rows and of the row
// above -- while the spins sit in LDS as two colour planes.  A pass reads the
// other plane, writes its own and ends at a barrier, so that global memory
// sees the inputs once, the saved spins (which the gradient needs) and the
// result: 8 B per attempt at most instead of the 32 (forward) and 76
// (backward) of a launch per pass, which re-reads spins and couplings.  Bound
// by VALU work: two exponentials, a division and Philox, about 90
// lane-instructions an attempt forward, 130 backward.
namespace {

struct ResLane {
    int y0, j, G, W;      // first row, span, spans per row, plane row length
    int o, ou, od;        // plane offsets of the span in rows y0, y0 - 1, y0 + NI
    int dL, dR;           // from a span to the columns left and right of it
    bool in;

    // Opaque offsets: a row's addresses are a few additions from these, and
    // worked out in the row; kept over the loop of passes instead, those of
    // all rows and passes would take the registers that the rows' state needs.
    __device__ __forceinline__ ResLane here() const {
        ResLane l = *this;
        asm volatile("" : "+v"(l.o), "+v"(l.ou), "+v"(l.od), "+v"(l.dL), "+v"(l.dR));
        return l;
    }
};

template <int NI>
__device__ __forceinline__ ResLane res_lane(const DmcArgs& a) {
    ResLane L;
    L.G = a.Lx >> 3;
    L.W = a.Lx >> 1;
    const int rows = a.Ly / NI;
    L.in = (int)threadIdx.x < rows * L.G;
    const int t = L.in ? (int)threadIdx.x : 0;
    const int rg = t / L.G;
    L.j = t - rg * L.G;
    L.y0 = rg * NI;
    L.o = L.y0 * L.W + 4 * L.j;
    L.ou = (L.y0 == 0 ? a.Ly - 1 : L.y0 - 1) * L.W + 4 * L.j;
    L.od = (L.y0 + NI == a.Ly ? 0 : L.y0 + NI) * L.W + 4 * L.j;
    L.dL = L.j == 0 ? L.W - 1 : -1;
    L.dR = L.j + 1 == L.G ? -4 * L.j : 4;
    return L;
}

__device__ __forceinline__ void unpack8(const Row8& r, float* v) {
    v[0] = r.a.x; v[1] = r.a.y; v[2] = r.a.z; v[3] = r.a.w;
    v[4] = r.b.x; v[5] = r.b.y; v[6] = r.b.z; v[7] = r.b.w;
}

__device__ __forceinline__ void store8(float* p, const float* v) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}

// jx[r][0] the bond left of the span, jx[r][1 + x] bond x
template <int NI>
__device__ __forceinline__ void res_jx(const DmcArgs& a, const ResLane& L, size_t off,
                                       float (&jx)[NI][9]) {
    const float* Jx = a.Jx + off;
    const int x0 = 8 * L.j, xl = L.j == 0 ? a.Lx - 1 : x0 - 1;
#pragma unroll
    for (int r = 0; r < NI; ++r) {
        const uint32_t row = (uint32_t)(L.y0 + r) * a.Lx;
        jx[r][0] = Jx[row + xl];
        unpack8(ld8(Jx + row + x0), &jx[r][1]);
    }
}

// jy[r] the bonds above row y0 + r
template <int NI>
__device__ __forceinline__ void res_jy(const DmcArgs& a, const ResLane& L, size_t off,
                                       float (&jy)[NI + 1][8]) {
    const float* Jy = a.Jy + off;
    const int x0 = 8 * L.j;
#pragma unroll
    for (int r = 0; r < NI; ++r)
        unpack8(ld8(Jy + (uint32_t)(L.y0 + r) * a.Lx + x0), &jy[r + 1][0]);
    const uint32_t up = (uint32_t)(L.y0 == 0 ? a.Ly - 1 : L.y0 - 1) * a.Lx;
    unpack8(ld8(Jy + up + x0), &jy[0][0]);
}

// The lane's rows of a natural-order lattice into the planes and back
template <int NI>
__device__ __forceinline__ void res_load(const float* s, int Lx, const ResLane& L, float* sp,
                                         int plane) {
#pragma unroll
    for (int r = 0; r < NI; ++r) {
        const Row8 v = ld8(s + (uint32_t)(L.y0 + r) * Lx + 8 * L.j);
        float* q = sp + L.o + r * L.W;
        *reinterpret_cast<float4*>(q + (r & 1) * plane) = make_float4(v.a.x, v.a.z, v.b.x, v.b.z);
        *reinterpret_cast<float4*>(q + (1 - (r & 1)) * plane) =
            make_float4(v.a.y, v.a.w, v.b.y, v.b.w);
    }
}

template <int NI>
__device__ __forceinline__ void res_store(float* s, int Lx, const ResLane& L, const float* sp,
                                          int plane) {
#pragma unroll
    for (int r = 0; r < NI; ++r) {
        const float* q = sp + L.o + r * L.W;
        const float4 e = *reinterpret_cast<const float4*>(q + (r & 1) * plane);
        const float4 o = *reinterpret_cast<const float4*>(q + (1 - (r & 1)) * plane);
        float* d = s + (uint32_t)(L.y0 + r) * Lx + 8 * L.j;
        *reinterpret_cast<float4*>(d) = make_float4(e.x, o.x, e.y, o.y);
        *reinterpret_cast<float4*>(d + 4) = make_float4(e.z, o.z, e.w, o.w);
    }
}

// A row's values in the other plane around its four own sites: row y itself
// with the value beyond the span on the side PAR reaches, rows y + 1 and
// y - 1
struct ResNb {
    float m[4], e, d[4], u[4];
};

template <int NI, int PAR, int R>
__device__ __forceinline__ ResNb res_nb(const float* p, const ResLane& L) {
    ResNb n;
    const int o = L.o + R * L.W;
    const float4 m = *reinterpret_cast<const float4*>(p + o);
    const float4 u = *reinterpret_cast<const float4*>(p + (R == 0 ? L.ou : o - L.W));
    const float4 d = *reinterpret_cast<const float4*>(p + (R == NI - 1 ? L.od : o + L.W));
    n.e = p[o + (PAR ? L.dR : L.dL)];
    n.m[0] = m.x; n.m[1] = m.y; n.m[2] = m.z; n.m[3] = m.w;
    n.u[0] = u.x; n.u[1] = u.y; n.u[2] = u.z; n.u[3] = u.w;
    n.d[0] = d.x; n.d[1] = d.y; n.d[2] = d.z; n.d[3] = d.w;
    return n;
}

// horizontal neighbours of own site u (column 2u + PAR of the span)
template <int PAR>
__device__ __forceinline__ float nb_left(const ResNb& n, int u) {
    return PAR ? n.m[u] : (u == 0 ? n.e : n.m[u > 0 ? u - 1 : 0]);
}
template <int PAR>
__device__ __forceinline__ float nb_right(const ResNb& n, int u) {
    return PAR ? (u == 3 ? n.e : n.m[u < 3 ? u + 1 : 3]) : n.m[u];
}

template <int NI, int C, int R>
__device__ __forceinline__ void res_fwd_row(const DmcArgs& a, const ResLane& L, float* sp, int plane,
                                            uint32_t p, uint32_t rid, float* save,
                                            const float (&jx)[NI][9], const float (&jy)[NI + 1][8]) {
    constexpr int PAR = (R + C) & 1;
    const int o = L.o + R * L.W, b = o >> 2;  // Philox block: within-colour index / 4
    float* own = sp + C * plane + o;
    const ResNb n = res_nb<NI, PAR, R>(sp + (1 - C) * plane, L);
    const float4 so = *reinterpret_cast<const float4*>(own);
    uint32_t w[4];
    philox4x32_10((uint32_t)b, p, rid, kTagDmc, a.key0, a.key1, w);
    float snew[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int x = 2 * u + PAR;
        const float sv = el4(so, u);
        const DmcUpd Q = dmc_update(sv, jx[R][x + 1], nb_right<PAR>(n, u), jx[R][x],
                                    nb_left<PAR>(n, u), jy[R + 1][x], n.d[u], jy[R][x], n.u[u],
                                    a.beta, a.alpha, a.h, w[u]);
        snew[u] = sv * (1.0f - 2.0f * Q.q);
    }
    *reinterpret_cast<float4*>(save + o) = so;
    *reinterpret_cast<float4*>(own) = make_float4(snew[0], snew[1], snew[2], snew[3]);
}

template <int NI, int C>
__device__ __forceinline__ void res_fwd_pass(const DmcArgs& a, const ResLane& L, float* sp, int plane,
                                             uint32_t p, uint32_t rid, float* save,
                                             const float (&jx)[NI][9], const float (&jy)[NI + 1][8]) {
    res_fwd_row<NI, C, 0>(a, L, sp, plane, p, rid, save, jx, jy);
    res_fwd_row<NI, C, 1>(a, L, sp, plane, p, rid, save, jx, jy);
    if constexpr (NI == 4) {
        res_fwd_row<NI, C, 2>(a, L, sp, plane, p, rid, save, jx, jy);
        res_fwd_row<NI, C, 3>(a, L, sp, plane, p, rid, save, jx, jy);
    }
}

// What a lane carries through the replay: the horizontal couplings, the
// gradients of all its bonds (those left of the span and above the first row
// are shares that go to the lanes that own the bonds at the end) and the
// adjoints g.  (The vertical couplings too would be 40 more registers of the
// 256 a lane of eight waves has at NI = 4: they sit in LDS, in colour planes
// like the spins.)
template <int NI>
struct ResGrad {
    float jx[NI][9], gx[NI][9], gy[NI + 1][8], g[NI][8];
};

template <int NI, int C, int R>
__device__ __forceinline__ void res_bwd_row(const DmcArgs& a, const ResLane& L0, float* sp,
                                            const float* jp, const float* tp, int plane, uint32_t p,
                                            uint32_t rid, bool first, const float4& sold4,
                                            float (&tv)[NI][4], ResGrad<NI>& S) {
    constexpr int PAR = (R + C) & 1;
    const ResLane L = L0.here();
    const int o = L.o + R * L.W, b = o >> 2;
    const ResNb n = res_nb<NI, PAR, R>(sp + (1 - C) * plane, L);
    const ResNb t4 = res_nb<NI, PAR, R>(tp, L);
    const float4 jd4 = *reinterpret_cast<const float4*>(jp + C * plane + o);
    const float4 ju4 =
        *reinterpret_cast<const float4*>(jp + (1 - C) * plane + (R == 0 ? L.ou : o - L.W));
    uint32_t w[4];
    philox4x32_10((uint32_t)b, p, rid, kTagDmc, a.key0, a.key1, w);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int x = 2 * u + PAR;
        const float sv = el4(sold4, u);
        const float jr = S.jx[R][x + 1], jl = S.jx[R][x], jd = el4(jd4, u), ju = el4(ju4, u);
        const float sr = nb_right<PAR>(n, u), sl = nb_left<PAR>(n, u);
        const DmcUpd Q = dmc_update(sv, jr, sr, jl, sl, jd, n.d[u], ju, n.u[u], a.beta, a.alpha,
                                    a.h, w[u]);
        float av = S.g[R][x];
        if (!first)
            av += jr * nb_right<PAR>(t4, u) + jl * nb_left<PAR>(t4, u) + jd * t4.d[u] + ju * t4.u[u];
        const float wq = 4.0f * a.alpha * a.beta * Q.q * (1.0f - Q.q) * Q.P;
        S.g[R][x] = av * ((1.0f - 2.0f * Q.q) + wq * sv * Q.hloc);
        const float t = av * wq * sv * sv;
        tv[R][u] = t;
        S.gx[R][x + 1] += t * sr;
        S.gx[R][x] += t * sl;
        S.gy[R + 1][x] += t * n.d[u];
        S.gy[R][x] += t * n.u[u];
    }
    *reinterpret_cast<float4*>(sp + C * plane + o) = sold4;
    // rows stay in sequence: interleaved, their temporaries do not fit
    __builtin_amdgcn_sched_barrier(0);
}

// One pass of the replay; nx holds the saved spins of its first row on entry
// and those of the next pass's first row on exit (each row's load is issued a
// row ahead), next the saved plane of the next pass (or this one's, if none).
template <int NI, int C>
__device__ __forceinline__ void res_bwd_pass(const DmcArgs& a, const ResLane& L, float* sp,
                                             const float* jp, const float* tp, int plane, uint32_t p,
                                             uint32_t rid, bool first, const float* save,
                                             const float* next, float4& nx, float (&tv)[NI][4],
                                             ResGrad<NI>& S) {
    const int o = L.o, st = L.W;
    float4 c = nx;
    nx = *reinterpret_cast<const float4*>(save + o + st);
    res_bwd_row<NI, C, 0>(a, L, sp, jp, tp, plane, p, rid, first, c, tv, S);
    c = nx;
    nx = *reinterpret_cast<const float4*>(NI == 4 ? save + o + 2 * st : next + o);
    res_bwd_row<NI, C, 1>(a, L, sp, jp, tp, plane, p, rid, first, c, tv, S);
    if constexpr (NI == 4) {
        c = nx;
        nx = *reinterpret_cast<const float4*>(save + o + 3 * st);
        res_bwd_row<NI, C, 2>(a, L, sp, jp, tp, plane, p, rid, first, c, tv, S);
        c = nx;
        nx = *reinterpret_cast<const float4*>(next + o);
        res_bwd_row<NI, C, 3>(a, L, sp, jp, tp, plane, p, rid, first, c, tv, S);
    }
}

// The t of a pass into its plane: one plane serves both colours, since a pass
// has read the previous one's (a barrier apart) before it writes its own.
template <int NI>
__device__ __forceinline__ void res_put_t(const ResLane& L, float* tp, const float (&tv)[NI][4]) {
#pragma unroll
    for (int r = 0; r < NI; ++r)
        *reinterpret_cast<float4*>(tp + L.o + r * L.W) =
            make_float4(tv[r][0], tv[r][1], tv[r][2], tv[r][3]);
}

// the t J terms of the last replayed pass (colour 0) on the colour-1 sites
template <int NI, int R>
__device__ __forceinline__ void res_gather_row(const DmcArgs& a, const ResLane& L, const float* jp,
                                               const float* tp, int plane, ResGrad<NI>& S) {
    constexpr int PAR = (R + 1) & 1;
    const int o = L.o + R * L.W;
    const ResNb t4 = res_nb<NI, PAR, R>(tp, L);
    const float4 jd4 = *reinterpret_cast<const float4*>(jp + plane + o);
    const float4 ju4 = *reinterpret_cast<const float4*>(jp + (R == 0 ? L.ou : o - L.W));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int x = 2 * u + PAR;
        S.g[R][x] += S.jx[R][x + 1] * nb_right<PAR>(t4, u) + S.jx[R][x] * nb_left<PAR>(t4, u) +
                     el4(jd4, u) * t4.d[u] + el4(ju4, u) * t4.u[u];
    }
}

}  // namespace

template <int NI>
__global__ void __launch_bounds__(1024) k_dmc_resident_fwd(DmcArgs a, uint32_t p0, int n_sweeps,
                                                           float* save) {
    extern __shared__ __align__(16) float lds[];
    const int plane = a.Ly * (a.Lx >> 1);
    const int r = (int)blockIdx.x;
    const size_t off = (size_t)r * a.Lx * a.Ly, step = (size_t)a.R * plane;
    const ResLane L = res_lane<NI>(a);
    const uint32_t rid = a.rid0 + (uint32_t)r;
    float jx[NI][9], jy[NI + 1][8];
    res_jx<NI>(a, L, off, jx);
    res_jy<NI>(a, L, off, jy);
    if (L.in) res_load<NI>(a.s_in + off, a.Lx, L, lds, plane);
    __syncthreads();
    float* sv = save + (size_t)r * plane;
    for (int i = 0; i < n_sweeps; ++i) {
        const uint32_t p = p0 + 2u * (uint32_t)i;
        if (L.in) res_fwd_pass<NI, 0>(a, L, lds, plane, p, rid, sv, jx, jy);
        __syncthreads();
        if (L.in) res_fwd_pass<NI, 1>(a, L, lds, plane, p + 1u, rid, sv + step, jx, jy);
        __syncthreads();
        sv += 2 * step;
    }
    if (L.in) {
        res_store<NI>(a.s + off, a.Lx, L, lds, plane);
        if (a.s_copy) res_store<NI>(a.s_copy + off, a.Lx, L, lds, plane);
    }
}

// Dynamic LDS: two planes of the spins, two of the vertical couplings, one of
// t = dL/dhloc.
template <int NI>
__global__ void __launch_bounds__(512) k_dmc_resident_bwd(DmcArgs a, uint32_t p0, int n_sweeps,
                                                          const float* save, const float* g,
                                                          float* gs, float* gJx, float* gJy,
                                                          int fresh) {
    extern __shared__ __align__(16) float lds[];
    const int plane = a.Ly * (a.Lx >> 1), Lx = a.Lx;
    float* jp = lds + 2 * plane;
    float* tp = lds + 4 * plane;
    const int r = (int)blockIdx.x;
    const size_t off = (size_t)r * Lx * a.Ly, step = (size_t)a.R * plane;
    const ResLane L = res_lane<NI>(a);
    const uint32_t rid = a.rid0 + (uint32_t)r;
    ResGrad<NI> S;
    res_jx<NI>(a, L, off, S.jx);
#pragma unroll
    for (int q = 0; q < NI; ++q) {
        const uint32_t o = (uint32_t)(L.y0 + q) * Lx + 8 * L.j;
        S.gx[q][0] = 0.f;
        if (fresh) {
#pragma unroll
            for (int x = 0; x < 8; ++x) S.gx[q][1 + x] = S.gy[q + 1][x] = 0.f;
        } else {
            unpack8(ld8(gJx + off + o), &S.gx[q][1]);
            unpack8(ld8(gJy + off + o), &S.gy[q + 1][0]);
        }
        unpack8(ld8(g + off + o), &S.g[q][0]);
    }
#pragma unroll
    for (int x = 0; x < 8; ++x) S.gy[0][x] = 0.f;
    if (L.in) {
        res_load<NI>(a.s_in + off, Lx, L, lds, plane);
        res_load<NI>(a.Jy + off, Lx, L, jp, plane);
    }
    const float* sv = save + (size_t)(2 * n_sweeps - 1) * step + (size_t)r * plane;
    float4 nx = *reinterpret_cast<const float4*>(sv + L.o);
    float tv[NI][4];
    __syncthreads();
    for (int i = n_sweeps - 1; i >= 0; --i) {
        const uint32_t p = p0 + 2u * (uint32_t)i;
        if (L.in)
            res_bwd_pass<NI, 1>(a, L, lds, jp, tp, plane, p + 1u, rid, i == n_sweeps - 1, sv,
                                sv - step, nx, tv, S);
        __syncthreads();
        if (L.in) res_put_t<NI>(L, tp, tv);
        __syncthreads();
        sv -= step;
        if (L.in)
            res_bwd_pass<NI, 0>(a, L, lds, jp, tp, plane, p, rid, false, sv,
                                i > 0 ? sv - step : sv, nx, tv, S);
        __syncthreads();
        if (L.in) res_put_t<NI>(L, tp, tv);
        __syncthreads();
        sv -= step;
    }
    if (L.in) {
        res_gather_row<NI, 0>(a, L, jp, tp, plane, S);
        res_gather_row<NI, 1>(a, L, jp, tp, plane, S);
        if constexpr (NI == 4) {
            res_gather_row<NI, 2>(a, L, jp, tp, plane, S);
            res_gather_row<NI, 3>(a, L, jp, tp, plane, S);
        }
        if (!fresh) res_store<NI>(a.s + off, Lx, L, lds, plane);
    }
    __syncthreads();  // the planes are free: shares of other lanes' bonds
    const int lane = (int)threadIdx.x;
    if (L.in) {
        store8(lds + 8 * lane, S.gy[0]);
#pragma unroll
        for (int q = 0; q < NI; ++q) tp[NI * lane + q] = S.gx[q][0];
    }
    __syncthreads();
    if (!L.in) return;
    const int rows = a.Ly / NI, rg = L.y0 / NI;
    const int below = (rg + 1 == rows ? 0 : rg + 1) * L.G + L.j;
    const int right = rg * L.G + (L.j + 1 == L.G ? 0 : L.j + 1);
#pragma unroll
    for (int x = 0; x < 8; ++x) S.gy[NI][x] += lds[8 * below + x];
#pragma unroll
    for (int q = 0; q < NI; ++q) {
        const uint32_t o = (uint32_t)(L.y0 + q) * Lx + 8 * L.j;
        S.gx[q][8] += tp[NI * right + q];
        store8(gJx + off + o, &S.gx[q][1]);
        store8(gJy + off + o, &S.gy[q + 1][0]);
        store8(gs + off + o, &S.g[q][0]);
    }
}

namespace {

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

// Lanes of the resident form with NI rows a lane, or 0 where it does not fit or is the
// slower.  Lattices up to 2^14 sites (8-column spans; the aligned buffers of the span
// kernels).  One workgroup a replica, so that few replicas leave the chip to a launch per
// pass: the forms below take them from a number of sites of all replicas on, where both
// were measured equal (us of 20 sweeps, resident and a launch per pass).
// Forward: 2 rows a lane, up to 1024 lanes; beyond 768 (a fourth wave a SIMD) from 2^19
// sites: 128 x 128, 1 replica 142 and 119, 24 144 and 136, 32 144 and 144, 64 144 and
// 199; 112 x 128, 32 replicas 147 and 140, 48 146 and 168; 96 x 128 at any number 113 to
// 118 and 117 to 236.
// Backward: 2 rows up to 512 lanes (2^13 sites), 4 above, where the state of a lane fills
// 256 registers, from 400000 sites: 96 x 96, 32 replicas 273 and 244, 48 274 and 280;
// 128 x 128, 24 replicas 268 and 273, 64 274 and 449.
// 256 replicas of 128 x 128, 10 sweeps: forward 297 -> 95 us, backward 811 -> 203; 64 x
// 64, 4 replicas, with the calls around it: forward 126 -> 60, backward 212 -> 103.
// Separate inputs and outputs spare the caller four copies and two fills of its arrays
// (16 MB each there: 40 us).
int res_lanes(const DmcArgs& a, int NI, int max_lanes, int any_lanes, int64_t min_sites) {
    if (a.Ly % NI != 0) return 0;
    const int64_t lanes = (int64_t)(a.Ly / NI) * (a.Lx >> 3);
    if (lanes > any_lanes && (int64_t)a.R * a.Lx * a.Ly < min_sites) return 0;
    return lanes <= max_lanes ? (int)lanes : 0;
}

template <class F>
hipError_t res_launch(F fn, const DmcArgs& a, int lanes, size_t lds, void** args, hipStream_t s) {
    hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    return hipLaunchKernel((const void*)fn, dim3(a.R), dim3((lanes + 63) & ~63), args, lds, s);
}

}  // namespace

hipError_t launch_dmc_forward(const DmcArgs& a, uint64_t t0, int n_sweeps, float* save,
                              hipStream_t s) {
    const int n_sites = a.Ly * (a.Lx >> 1);
    const bool v8 = (a.Lx & 7) == 0 && aligned16(a.s) && aligned16(a.s_in) &&
                    aligned16(a.s_copy) && aligned16(a.Jx) && aligned16(a.Jy) && aligned16(save);
    const size_t bytes = sizeof(float) * a.R * a.Lx * a.Ly;
    const int n_blocks = (n_sites + 3) >> 2;
    if (const int lanes = v8 ? res_lanes(a, 2, 1024, 768, (int64_t)1 << 19) : 0) {
        DmcArgs b = a;
        uint32_t p0 = (uint32_t)(2 * t0);
        void* args[] = {&b, &p0, &n_sweeps, &save};
        return res_launch(k_dmc_resident_fwd<2>, a, lanes, (size_t)8 * n_sites, args, s);
    }
    hipError_t e = hipSuccess;
    if (a.s_in != a.s) e = hipMemcpyAsync(a.s, a.s_in, bytes, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return e;
    const dim3 grid((n_blocks + 255) / 256, a.R), block(256);
    for (int i = 0; i < n_sweeps; ++i)
        for (int c = 0; c < 2; ++c) {
            const uint32_t p = (uint32_t)(2 * (t0 + (uint64_t)i) + (uint64_t)c);
            float* sv = save + (size_t)(2 * i + c) * a.R * n_sites;
            if (v8)
                hipLaunchKernelGGL(k_dmc_pass8, grid, block, 0, s, a, c, p, sv);
            else
                hipLaunchKernelGGL(k_dmc_pass, grid, block, 0, s, a, c, p, sv);
        }
    e = hipGetLastError();
    if (e == hipSuccess && a.s_copy)
        e = hipMemcpyAsync(a.s_copy, a.s, bytes, hipMemcpyDeviceToDevice, s);
    return e;
}

hipError_t launch_dmc_backward(const DmcArgs& a, uint64_t t0, int n_sweeps, const float* save,
                               const float* g, float* gs, float* gJx, float* gJy, float* work,
                               bool fresh, hipStream_t s) {
    const int n_sites = a.Ly * (a.Lx >> 1);
    const size_t plane = (size_t)a.R * n_sites;
    const bool v8 = (a.Lx & 7) == 0 && aligned16(a.s) && aligned16(a.s_in) && aligned16(a.Jx) &&
                    aligned16(a.Jy) && aligned16(save) && aligned16(g) && aligned16(gs) && aligned16(gJx) && aligned16(gJy) &&
                    aligned16(work);
    const int n_blocks = (n_sites + 3) >> 2;
    {
        const int l2 = v8 && n_sweeps > 0 ? res_lanes(a, 2, 512, 512, 0) : 0;
        const int l4 = v8 && n_sweeps > 0 && l2 == 0 ? res_lanes(a, 4, 512, 0, 400000) : 0;
        DmcArgs b = a;
        uint32_t p0 = (uint32_t)(2 * t0);
        int fr = fresh ? 1 : 0;
        void* args[] = {&b, &p0, &n_sweeps, &save, &g, &gs, &gJx, &gJy, &fr};
        if (l2) return res_launch(k_dmc_resident_bwd<2>, a, l2, (size_t)20 * n_sites, args, s);
        if (l4) return res_launch(k_dmc_resident_bwd<4>, a, l4, (size_t)20 * n_sites, args, s);
    }
    hipError_t e = hipSuccess;
    if (fresh) {  // the passes below work in place
        const size_t n = 2 * plane;
        e = hipMemcpyAsync(a.s, a.s_in, sizeof(float) * n, hipMemcpyDeviceToDevice, s);
        if (e == hipSuccess && gs != g)
            e = hipMemcpyAsync(gs, g, sizeof(float) * n, hipMemcpyDeviceToDevice, s);
        if (e == hipSuccess) e = launch_fill_i32(reinterpret_cast<int32_t*>(gJx), n, 0, s);
        if (e == hipSuccess) e = launch_fill_i32(reinterpret_cast<int32_t*>(gJy), n, 0, s);
        if (e != hipSuccess) return e;
    }
    const dim3 grid((n_blocks + 255) / 256, a.R), gridg((n_sites + 255) / 256, a.R), block(256);
    // pass m = 2 i + c writes its t to plane m & 1 and folds in the t of
    // pass m + 1 from the other plane
    for (int m = 2 * n_sweeps - 1; m >= 0; --m) {
        const int i = m >> 1, c = m & 1;
        const uint32_t p = (uint32_t)(2 * (t0 + (uint64_t)i) + (uint64_t)c);
        const float* sv = save + (size_t)m * plane;
        const float* tin = m == 2 * n_sweeps - 1 ? nullptr : work + (size_t)((m + 1) & 1) * plane;
        float* tout = work + (size_t)(m & 1) * plane;
        if (v8)
            hipLaunchKernelGGL(k_dmc_back8, grid, block, 0, s, a, c, p, sv, gs, gJx, gJy,
                               tin, tout);
        else
            hipLaunchKernelGGL(k_dmc_back, grid, block, 0, s, a, c, p, sv, gs, gJx, gJy, tin,
                               tout);
    }
    if (n_sweeps > 0)  // pass 0 (colour 0): its t reach the colour-1 sites
        hipLaunchKernelGGL(k_dmc_gather, gridg, block, 0, s, a, 0, gs, work);
    return hipGetLastError();
}

}  // namespace spinmc
