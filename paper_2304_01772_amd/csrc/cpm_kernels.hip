// Cellular Potts model (Eq. (3)) copy-attempt kernels for gfx950.
//
// Cell ids are int32 in natural row-major layout.  The Moore neighbourhood
// has range one in both axes, so a 2x2 sublattice colouring
// c = 2 (y & 1) + (x & 1) makes the sites of one colour independent (the
// colouring criterion of the Related-Work section: no site interacts with
// another site of its own colour); a Monte Carlo step is the four colour
// passes in order.  Each attempt picks a target site and one of its eight
// neighbours (Methods, Cellular Potts model), and copies the neighbour's id
// through the Algorithm-1 test.  Energies are integers in a fixed-point
// scale S; the area term reads a snapshot of the cell areas taken at the
// start of the pass (so the outcome does not depend on the order in which
// the sites of one pass are visited), and accepted copies update the areas
// with integer atomics, which commute.  The streamed passes keep the
// snapshot without a copy launch: pass P reads it as S[P & 1] + D[(P-1) % 3]
// (the previous snapshot plus the previous pass's changes), adds its own
// changes into D[P % 3], and on the side writes its snapshot to S[(P+1) & 1]
// and clears D[(P+1) % 3] for pass P + 1 (buffers no other pass of the
// launch touches).
#include "cpm_internal.hpp"

namespace spinmc {

namespace {
__device__ __forceinline__ int wrapc(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// The rotating snapshot / change buffers of pass P for cells at offset off.
struct PassAreas {
    const int32_t* s_rd;  // previous snapshot
    const int32_t* d_rd;  // previous pass's changes
    int32_t* d_wr;        // this pass's changes
};
__device__ __forceinline__ PassAreas pass_areas(const CpmArgs& a, uint64_t P, int off) {
    const size_t n = (size_t)a.total_cells;
    PassAreas r;
    r.s_rd = a.sbuf + (size_t)(P & 1u) * n + off;
    r.d_rd = a.dbuf + (size_t)((P + 2u) % 3u) * n + off;
    r.d_wr = a.dbuf + (size_t)(P % 3u) * n + off;
    return r;
}

// Side work of pass P, spread over the launch's threads: the snapshot it
// reads goes to S[(P+1) & 1] and D[(P+1) % 3] is cleared.
__device__ __forceinline__ void pass_rotate(const CpmArgs& a, uint64_t P) {
    const size_t n = (size_t)a.total_cells;
    const int32_t* s_rd = a.sbuf + (size_t)(P & 1u) * n;
    const int32_t* d_rd = a.dbuf + (size_t)((P + 2u) % 3u) * n;
    int32_t* s_wr = a.sbuf + (size_t)((P + 1u) & 1u) * n;
    int32_t* d_clr = a.dbuf + (size_t)((P + 1u) % 3u) * n;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        s_wr[i] = s_rd[i] + d_rd[i];
        d_clr[i] = 0;
    }
}
}  // namespace

__global__ void __launch_bounds__(256) k_cpm_pass(CpmArgs a, int c, int sweep_off) {
    extern __shared__ uint32_t lthr[];  // [2 * tab_n]: hi16 | lo16 of T(k), k = 1..K1-1
    __shared__ int32_t ljs[kMaxCpmTypes * kMaxCpmTypes];
    const TileDev T = a.tiles[blockIdx.x];
    const RepDev R = a.reps[T.rep];
    for (int i = threadIdx.x; i < 2 * R.tab_n; i += blockDim.x) lthr[i] = a.tab[R.tab_off + i];
    for (int i = threadIdx.x; i < R.n_types * R.n_types; i += blockDim.x)
        ljs[i] = a.js[R.js_off + i];
    __syncthreads();
    const uint64_t t = *a.t_base + (uint64_t)sweep_off;
    const uint64_t P = 4 * t + (uint64_t)c;
    const uint32_t p = (uint32_t)P;
    pass_rotate(a, P);
    const PassAreas pa = pass_areas(a, P, R.cell_off);
    const int cy = c >> 1, cx = c & 1;
    const int Lx = R.Lx, Ly = R.Ly, Wc = Lx >> 1, nt = R.n_types;
    int32_t* ids = a.lat + R.lat_off;
    const int8_t* ty = a.ctype + R.cell_off;
    const int32_t* A = a.target + R.cell_off;
    int32_t* area = pa.d_wr;
    const auto snap_of = [&](int i) -> int64_t { return (int64_t)pa.s_rd[i] + pa.d_rd[i]; };
    const int total = (T.rows >> 1) * Wc;
    for (int it = threadIdx.x; it < total; it += blockDim.x) {
        const int r = it / Wc;
        const int i = it - r * Wc;
        const int y = T.y0 + 2 * r + cy;
        const int x = 2 * i + cx;
        const uint32_t k = (uint32_t)((y >> 1) * Wc + i);
        uint32_t w[4];
        philox4x32_10(k >> 2, p, R.rid, kTagMain, a.key0, a.key1, w);
        const uint32_t word = w[k & 3u];
        const int jn = (int)(word & 7u);
        // Moore order (dy, dx): (-1,-1) (-1,0) (-1,1) (0,-1) (0,1) (1,-1) (1,0) (1,1)
        const int ndy = jn < 3 ? -1 : (jn < 5 ? 0 : 1);
        const int ndx = (jn == 0 || jn == 3 || jn == 5) ? -1 : ((jn == 1 || jn == 6) ? 0 : 1);
        const int ym = wrapc(y - 1, Ly), yp = wrapc(y + 1, Ly);
        const int xm = wrapc(x - 1, Lx), xp = wrapc(x + 1, Lx);
        const int s = ids[(size_t)y * Lx + x];
        const int tg = ids[(size_t)wrapc(y + ndy, Ly) * Lx + wrapc(x + ndx, Lx)];
        if (tg == s) continue;
        const int nb[8] = {ids[(size_t)ym * Lx + xm], ids[(size_t)ym * Lx + x],
                           ids[(size_t)ym * Lx + xp], ids[(size_t)y * Lx + xm],
                           ids[(size_t)y * Lx + xp], ids[(size_t)yp * Lx + xm],
                           ids[(size_t)yp * Lx + x], ids[(size_t)yp * Lx + xp]};
        const int ts = ty[s] * nt, tt = ty[tg] * nt;
        int kadh = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int m = nb[j];
            const int tm = ty[m];
            kadh += (tg != m) ? ljs[tt + tm] : 0;
            kadh -= (s != m) ? ljs[ts + tm] : 0;
        }
        int64_t karea = 0;
        if (tg != 0) karea += 2 * (snap_of(tg) - (int64_t)A[tg]) + 1;
        if (s != 0) karea += -2 * (snap_of(s) - (int64_t)A[s]) + 1;
        const int64_t kk = (int64_t)kadh + R.LS * karea;
        bool acc;
        if (kk <= 0) {
            acc = true;
        } else if (kk >= R.K0) {
            acc = false;
        } else {
            uint32_t hi = 0u, lo = 1u;  // T = 1 for K1 <= k < K0
            if (kk < (int64_t)R.K1) {
                hi = lthr[kk - 1];
                lo = lthr[R.tab_n + kk - 1];
            }
            const uint32_t rr = word >> 16;
            acc = rr < hi;
            if (rr == hi && lo != 0u) {
                uint32_t f[4];
                philox4x32_10(k, p, R.rid, kTagFallback, a.key0, a.key1, f);
                acc = (f[0] & 0xFFFFu) < lo;
            }
        }
        if (acc) {
            ids[(size_t)y * Lx + x] = tg;
            atomicAdd(&area[tg], 1);
            atomicAdd(&area[s], -1);
        }
    }
}

// The 5x5 neighbourhood (the Moore neighbourhood with its second shell):
// 24 neighbours in row-major order of (dy, dx) for both the adhesion sum and
// the copy source; the 3x3 sublattice c = 3 (y % 3) + x % 3 keeps the sites
// of one colour out of each other's neighbourhoods; pass p = 9t + c, within-
// colour index k = (y / 3) Lx/3 + x / 3.  The neighbour index is Lemire's
// multiply-shift of the low 16 bits of the main word into 24, and where
// that rejects (16 of the 65536 values) the 32-bit multiply-shift of word 1
// of the fallback block.
// The 5x5 copy attempt of site (y, x), within-colour index k, colour pass p:
// ty the cell types, sa(i) the pass-start area minus target of cell i (as
// int64); accepted copies update ids and area.
template <class SA>
__device__ __forceinline__ void cpm5_attempt(const CpmArgs& a, const RepDev& R, int32_t* ids,
                                             int32_t* area, int y, int x, uint32_t k, uint32_t p,
                                             const uint32_t* lthr, const int8_t* ty,
                                             const int32_t* ljs, SA sa) {
    const int Lx = R.Lx, Ly = R.Ly, nt = R.n_types;
    uint32_t w[4];
    philox4x32_10(k >> 2, p, R.rid, kTagMain, a.key0, a.key1, w);
    const uint32_t word = w[k & 3u];
    uint32_t f[4];
    bool have_f = false;
    const uint32_t l = (word & 0xFFFFu) * 24u;
    int jn = (int)(l >> 16);
    if ((l & 0xFFFFu) < 16u) {
        philox4x32_10(k, p, R.rid, kTagFallback, a.key0, a.key1, f);
        have_f = true;
        jn = (int)(((uint64_t)f[1] * 24u) >> 32);
    }
    // row-major offsets without the centre: jn < 12 lies before it
    const int jj = jn < 12 ? jn : jn + 1;
    const int ndy = jj / 5 - 2, ndx = jj % 5 - 2;
    int rows[5], cols[5];
#pragma unroll
    for (int d = 0; d < 5; ++d) {
        rows[d] = wrapc(y + d - 2, Ly) * Lx;
        cols[d] = wrapc(x + d - 2, Lx);
    }
    const int s = ids[(size_t)rows[2] + x];
    const int tg = ids[(size_t)wrapc(y + ndy, Ly) * Lx + wrapc(x + ndx, Lx)];
    if (tg == s) return;
    int nb[25];
#pragma unroll
    for (int dy = 0; dy < 5; ++dy)
#pragma unroll
        for (int dx = 0; dx < 5; ++dx) nb[dy * 5 + dx] = ids[(size_t)rows[dy] + cols[dx]];
    const int ts = ty[s] * nt, tt = ty[tg] * nt;
    int kadh = 0;
#pragma unroll
    for (int j = 0; j < 25; ++j) {
        if (j == 12) continue;  // the site itself
        const int m = nb[j];
        const int tm = ty[m];
        kadh += (tg != m) ? ljs[tt + tm] : 0;
        kadh -= (s != m) ? ljs[ts + tm] : 0;
    }
    int64_t karea = 0;
    if (tg != 0) karea += 2 * sa(tg) + 1;
    if (s != 0) karea += -2 * sa(s) + 1;
    const int64_t kk = (int64_t)kadh + R.LS * karea;
    bool acc;
    if (kk <= 0) {
        acc = true;
    } else if (kk >= R.K0) {
        acc = false;
    } else {
        uint32_t hi = 0u, lo = 1u;  // T = 1 for K1 <= k < K0
        if (kk < (int64_t)R.K1) {
            hi = lthr[kk - 1];
            lo = lthr[R.tab_n + kk - 1];
        }
        const uint32_t rr = word >> 16;
        acc = rr < hi;
        if (rr == hi && lo != 0u) {
            if (!have_f) philox4x32_10(k, p, R.rid, kTagFallback, a.key0, a.key1, f);
            acc = (f[0] & 0xFFFFu) < lo;
        }
    }
    if (acc) {
        ids[(size_t)rows[2] + x] = tg;
        atomicAdd(&area[tg], 1);
        atomicAdd(&area[s], -1);
    }
}

__global__ void __launch_bounds__(256) k_cpm_pass5(CpmArgs a, int c, int sweep_off) {
    extern __shared__ uint32_t lthr[];  // [2 * tab_n]: hi16 | lo16 of T(k), k = 1..K1-1
    __shared__ int32_t ljs[kMaxCpmTypes * kMaxCpmTypes];
    const TileDev T = a.tiles[blockIdx.x];
    const RepDev R = a.reps[T.rep];
    for (int i = threadIdx.x; i < 2 * R.tab_n; i += blockDim.x) lthr[i] = a.tab[R.tab_off + i];
    for (int i = threadIdx.x; i < R.n_types * R.n_types; i += blockDim.x)
        ljs[i] = a.js[R.js_off + i];
    __syncthreads();
    const uint64_t t = *a.t_base + (uint64_t)sweep_off;
    const uint64_t P = 9 * t + (uint64_t)c;
    const uint32_t p = (uint32_t)P;
    pass_rotate(a, P);
    const PassAreas pa = pass_areas(a, P, R.cell_off);
    const int cy = c / 3, cx = c - 3 * cy;
    const int Lx = R.Lx, Wc = Lx / 3;
    int32_t* ids = a.lat + R.lat_off;
    const int8_t* ty = a.ctype + R.cell_off;
    const int32_t* A = a.target + R.cell_off;
    int32_t* area = pa.d_wr;
    const int32_t* s_rd = pa.s_rd;
    const int32_t* d_rd = pa.d_rd;
    const auto sa = [=](int i) -> int64_t {
        return (int64_t)s_rd[i] + (int64_t)d_rd[i] - (int64_t)A[i];
    };
    const int total = (T.rows / 3) * Wc;
    for (int it = threadIdx.x; it < total; it += blockDim.x) {
        const int r = it / Wc;
        const int i = it - r * Wc;
        const int y = T.y0 + 3 * r + cy;
        const int x = 3 * i + cx;
        const uint32_t k = (uint32_t)((y / 3) * Wc + i);
        cpm5_attempt(a, R, ids, area, y, x, k, p, lthr, ty, ljs, sa);
    }
}

// The same pass with four consecutive same-colour sites of one row per lane
// (Lx a multiple of 8): their attempts share one Philox call (words 0..3 of
// counter k >> 2), their 3 x 9 id window comes in with six 16-byte loads and
// three halo loads, and the per-cell tables (type, pass-start area minus
// target) sit in LDS, so that a lane's attempts wait for one round of
// global loads.
__device__ __forceinline__ int sel8(const int (&v)[8], uint32_t j) {
    const int a0 = (j & 1u) ? v[1] : v[0], a1 = (j & 1u) ? v[3] : v[2];
    const int a2 = (j & 1u) ? v[5] : v[4], a3 = (j & 1u) ? v[7] : v[6];
    const int b0 = (j & 2u) ? a1 : a0, b1 = (j & 2u) ? a3 : a2;
    return (j & 4u) ? b1 : b0;
}

// The copy attempt of site x (id s, Moore neighbours nb in the order
// (dy, dx) = (-1,-1) (-1,0) (-1,1) (0,-1) (0,1) (1,-1) (1,0) (1,1)) with main
// word `word` (bits 0..2 the neighbour, bits 16..31 the prefix r of W) and
// within-colour index k (the fallback counter): the id to copy, or -1.
__device__ __forceinline__ int cpm_decide(const CpmArgs& a, const RepDev& R, const int (&nb)[8],
                                          int s, uint32_t word, uint32_t k, uint32_t p,
                                          const uint32_t* qthr, const int32_t* lsa,
                                          const int8_t* lty, const int32_t* ljs) {
    const int nt = R.n_types;
    const int tg = sel8(nb, word & 7u);
    if (tg == s) return -1;
    const int ts = lty[s] * nt, tt = lty[tg] * nt;
    int kadh = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int m = nb[j];
        const int tm = lty[m];
        kadh += (tg != m) ? ljs[tt + tm] : 0;
        kadh -= (s != m) ? ljs[ts + tm] : 0;
    }
    int64_t karea = 0;
    if (tg != 0) karea += 2 * (int64_t)lsa[tg] + 1;
    if (s != 0) karea += -2 * (int64_t)lsa[s] + 1;
    const int64_t kk = (int64_t)kadh + R.LS * karea;
    bool acc;
    if (kk <= 0) {
        acc = true;
    } else if (kk >= R.K0) {
        acc = false;
    } else {
        uint32_t hi = 0u, lo = 1u;  // T = 1 for K1 <= k < K0
        if (kk < (int64_t)R.K1) {
            hi = qthr[kk - 1];
            lo = qthr[R.tab_n + kk - 1];
        }
        const uint32_t rr = word >> 16;
        acc = rr < hi;
        if (rr == hi && lo != 0u) {
            uint32_t f[4];
            philox4x32_10(k, p, R.rid, kTagFallback, a.key0, a.key1, f);
            acc = (f[0] & 0xFFFFu) < lo;
        }
    }
    return acc ? tg : -1;
}

// ids / area: the replica's cell ids and live areas (global memory for the
// streamed pass, LDS for the resident kernel); rows y0 .. y0 + rows - 1.

// Per-cell tables of replica R into LDS for one pass of a tile: thresholds,
// adhesion, types and pass-start area minus target.  Each thread issues up
// to 4 items' loads before storing any, so that the tables arrive in one
// round of global loads.
__device__ __forceinline__ void cpm_stage(const CpmArgs& a, const RepDev& R, const PassAreas& pa,
                                          uint32_t* qthr, int32_t* lsa, int8_t* lty,
                                          int32_t* ljs) {
    const int ncell = R.q + 1;
    const int8_t* ty = a.ctype + R.cell_off;
    const int32_t* A = a.target + R.cell_off;
    const int nthr = blockDim.x;
    const int ntab = 2 * R.tab_n;
    for (int i0 = threadIdx.x; i0 < ntab; i0 += 4 * nthr) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * nthr;
            v[u] = i < ntab ? a.tab[R.tab_off + i] : 0u;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i0 + u * nthr < ntab) qthr[i0 + u * nthr] = v[u];
    }
    for (int i = threadIdx.x; i < R.n_types * R.n_types; i += nthr) ljs[i] = a.js[R.js_off + i];
    for (int i0 = threadIdx.x; i0 < ncell; i0 += 4 * nthr) {
        int32_t sv[4], av[4];
        int8_t tv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * nthr;
            const bool in = i < ncell;
            sv[u] = in ? pa.s_rd[i] + pa.d_rd[i] : 0;
            av[u] = in ? A[i] : 0;
            tv[u] = in ? ty[i] : (int8_t)0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * nthr;
            if (i < ncell) {
                lsa[i] = sv[u] - av[u];
                lty[i] = tv[u];
            }
        }
    }
}


// One quad's inputs: its 3 x 9 id window (rows y - 1, y, y + 1; the halo
// column on the side of colour CX) and its Philox block.
struct QuadIn {
    int win[3][9];
    uint32_t w[4];
    int y, x0;
    uint32_t kq;
};

// Loads of quad `it` of the colour-(2 cy + CX) sites of rows y0 ..: six
// 16-byte loads, three halo loads and the Philox block (k >> 2 of the four
// sites); nothing here reads the staged tables.
template <int CX>
__device__ __forceinline__ void quad_load(const CpmArgs& a, const RepDev& R, const int32_t* ids,
                                          int y0, int cy, uint32_t p, int it, QuadIn& q) {
    const int Lx = R.Lx, Ly = R.Ly, Q = Lx >> 3;
    const int r = it / Q;
    const int qi = it - r * Q;
    q.y = y0 + 2 * r + cy;
    q.x0 = 8 * qi;
    q.kq = (uint32_t)((q.y >> 1) * Q + qi);
    const int yr[3] = {wrapc(q.y - 1, Ly), q.y, wrapc(q.y + 1, Ly)};
    const int xh = CX == 0 ? wrapc(q.x0 - 1, Lx) : wrapc(q.x0 + 8, Lx);
#pragma unroll
    for (int rr = 0; rr < 3; ++rr) {
        const int32_t* row = ids + (size_t)yr[rr] * Lx;
        const int4 u = *reinterpret_cast<const int4*>(row + q.x0);
        const int4 v = *reinterpret_cast<const int4*>(row + q.x0 + 4);
        const int h = row[xh];
        constexpr int o = CX == 0 ? 1 : 0;
        q.win[rr][o + 0] = u.x;
        q.win[rr][o + 1] = u.y;
        q.win[rr][o + 2] = u.z;
        q.win[rr][o + 3] = u.w;
        q.win[rr][o + 4] = v.x;
        q.win[rr][o + 5] = v.y;
        q.win[rr][o + 6] = v.z;
        q.win[rr][o + 7] = v.w;
        q.win[rr][CX == 0 ? 0 : 8] = h;
    }
    philox4x32_10(q.kq, p, R.rid, kTagMain, a.key0, a.key1, q.w);
}

// The quad's four attempts (site 2u + CX of the quad is word u) and, on
// acceptance, the id update and the area changes (LDS atomics into the
// workgroup's per-cell sums).
template <int CX>
__device__ __forceinline__ void quad_decide(const CpmArgs& a, const RepDev& R, int32_t* ids,
                                            int32_t* area, uint32_t p, const QuadIn& q,
                                            const uint32_t* qthr, const int32_t* lsa,
                                            const int8_t* lty, const int32_t* ljs) {
    const int Lx = R.Lx;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        // Moore order (dy, dx): (-1,-1) (-1,0) (-1,1) (0,-1) (0,1) (1,-1) (1,0) (1,1)
        const int nb[8] = {q.win[0][2 * u], q.win[0][2 * u + 1], q.win[0][2 * u + 2],
                           q.win[1][2 * u], q.win[1][2 * u + 2],
                           q.win[2][2 * u], q.win[2][2 * u + 1], q.win[2][2 * u + 2]};
        const int s = q.win[1][2 * u + 1];
        const int tg = cpm_decide(a, R, nb, s, q.w[u], 4u * q.kq + (uint32_t)u, p, qthr, lsa, lty,
                                  ljs);
        if (tg >= 0) {
            ids[(size_t)q.y * Lx + q.x0 + 2 * u + CX] = tg;
            atomicAdd(&area[tg], 1);
            atomicAdd(&area[s], -1);
        }
    }
}

// A lane's first quad is loaded (window and Philox block) before the
// per-cell tables are staged, so that the two rounds of global loads
// overlap; the other quads of the lane follow the table barrier.  Area
// changes gather in LDS (one sum per cell of the replica) and go to the
// pass's change buffer as one global atomic per touched cell at the end:
// integer sums, so the buffer ends equal to one atomic per copy, with far
// fewer atomics on the cells' words.
template <int CX>
__device__ __forceinline__ void quad_pass(const CpmArgs& a, int c, int sweep_off,
                                          uint32_t* qthr, int32_t* lsa, int8_t* lty,
                                          int32_t* ljs, int32_t* ldel) {
    const TileDev T = a.tiles[blockIdx.x];
    const RepDev R = a.reps[T.rep];
    const uint64_t t = *a.t_base + (uint64_t)sweep_off;
    const uint64_t P = 4 * t + (uint64_t)c;
    const uint32_t p = (uint32_t)P;
    const PassAreas pa = pass_areas(a, P, R.cell_off);
    int32_t* ids = a.lat + R.lat_off;
    const int cy = c >> 1;
    const int total = (T.rows >> 1) * (R.Lx >> 3);
    const int it0 = (int)threadIdx.x;
    QuadIn q;
    if (it0 < total) quad_load<CX>(a, R, ids, T.y0, cy, p, it0, q);
    cpm_stage(a, R, pa, qthr, lsa, lty, ljs);
    pass_rotate(a, P);
    const int ncell = R.q + 1;
    for (int i = (int)threadIdx.x; i < ncell; i += (int)blockDim.x) ldel[i] = 0;
    __syncthreads();
    if (it0 < total) quad_decide<CX>(a, R, ids, ldel, p, q, qthr, lsa, lty, ljs);
    for (int it = it0 + (int)blockDim.x; it < total; it += blockDim.x) {
        quad_load<CX>(a, R, ids, T.y0, cy, p, it, q);
        quad_decide<CX>(a, R, ids, ldel, p, q, qthr, lsa, lty, ljs);
    }
    __syncthreads();
    for (int i = (int)threadIdx.x; i < ncell; i += (int)blockDim.x) {
        const int d = ldel[i];
        if (d != 0) atomicAdd(&pa.d_wr[i], d);
    }
}

// One lane per site (the "site" form of the quad pass): lane u of each
// group of four takes site 2u + CX of a quad, computes the quad's Philox
// block itself and keeps word u, loads its own 3 x 3 window and decides one
// attempt, so that a workgroup of 1024 lanes carries four times the
// attempts in flight of the quad form at the same tile, each lane's
// chain of table lookups a quarter as long.  Same decisions, same stores;
// area changes gather in LDS as in the quad form.
struct SiteIn {
    int nb[8];
    int s;
    uint32_t w;
    int y, x;
    uint32_t kq;
};

template <int CX>
__device__ __forceinline__ void site_load(const CpmArgs& a, const RepDev& R, const int32_t* ids,
                                          int y0, int cy, uint32_t p, int it, int u, SiteIn& q) {
    const int Lx = R.Lx, Ly = R.Ly, Q = Lx >> 3;
    const int r = it / Q;
    const int qi = it - r * Q;
    q.y = y0 + 2 * r + cy;
    q.x = 8 * qi + 2 * u + CX;
    q.kq = (uint32_t)((q.y >> 1) * Q + qi);
    const int yu = wrapc(q.y - 1, Ly), yd = wrapc(q.y + 1, Ly);
    const int xl = wrapc(q.x - 1, Lx), xr = wrapc(q.x + 1, Lx);
    const int32_t* ru = ids + (size_t)yu * Lx;
    const int32_t* ry = ids + (size_t)q.y * Lx;
    const int32_t* rd = ids + (size_t)yd * Lx;
    // Moore order (dy, dx): (-1,-1) (-1,0) (-1,1) (0,-1) (0,1) (1,-1) (1,0) (1,1)
    q.nb[0] = ru[xl];
    q.nb[1] = ru[q.x];
    q.nb[2] = ru[xr];
    q.nb[3] = ry[xl];
    q.nb[4] = ry[xr];
    q.nb[5] = rd[xl];
    q.nb[6] = rd[q.x];
    q.nb[7] = rd[xr];
    q.s = ry[q.x];
    uint32_t w[4];
    philox4x32_10(q.kq, p, R.rid, kTagMain, a.key0, a.key1, w);
    q.w = u == 0 ? w[0] : (u == 1 ? w[1] : (u == 2 ? w[2] : w[3]));
}

template <int CX>
__device__ __forceinline__ void site_pass(const CpmArgs& a, int c, int sweep_off,
                                          uint32_t* qthr, int32_t* lsa, int8_t* lty,
                                          int32_t* ljs, int32_t* ldel) {
    const TileDev T = a.tiles[blockIdx.x];
    const RepDev R = a.reps[T.rep];
    const uint64_t t = *a.t_base + (uint64_t)sweep_off;
    const uint64_t P = 4 * t + (uint64_t)c;
    const uint32_t p = (uint32_t)P;
    const PassAreas pa = pass_areas(a, P, R.cell_off);
    int32_t* ids = a.lat + R.lat_off;
    const int cy = c >> 1;
    const int total = (T.rows >> 1) * (R.Lx >> 3);  // quads of the tile
    const int u = (int)threadIdx.x & 3, qs = (int)blockDim.x >> 2;
    int it = (int)threadIdx.x >> 2;
    SiteIn q;
    if (it < total) site_load<CX>(a, R, ids, T.y0, cy, p, it, u, q);
    cpm_stage(a, R, pa, qthr, lsa, lty, ljs);
    pass_rotate(a, P);
    const int ncell = R.q + 1;
    for (int i = (int)threadIdx.x; i < ncell; i += (int)blockDim.x) ldel[i] = 0;
    __syncthreads();
    while (it < total) {
        const int tg = cpm_decide(a, R, q.nb, q.s, q.w, 4u * q.kq + (uint32_t)u, p, qthr, lsa,
                                  lty, ljs);
        if (tg >= 0) {
            ids[(size_t)q.y * R.Lx + q.x] = tg;
            atomicAdd(&ldel[tg], 1);
            atomicAdd(&ldel[q.s], -1);
        }
        it += qs;
        if (it < total) site_load<CX>(a, R, ids, T.y0, cy, p, it, u, q);
    }
    __syncthreads();
    for (int i = (int)threadIdx.x; i < ncell; i += (int)blockDim.x) {
        const int d = ldel[i];
        if (d != 0) atomicAdd(&pa.d_wr[i], d);
    }
}

__global__ void __launch_bounds__(256) k_cpm_pass_quad(CpmArgs a, int c, int sweep_off,
                                                       int tab_lds_bytes, int cell_cap) {
    // dynamic LDS: [T hi | T lo] (tab_lds_bytes) | snap - A (int32) | type (int8) |
    // area changes of the pass (int32); cell_cap is a multiple of 16
    extern __shared__ __align__(16) uint8_t dyn[];
    uint32_t* qthr = reinterpret_cast<uint32_t*>(dyn);
    int32_t* lsa = reinterpret_cast<int32_t*>(dyn + tab_lds_bytes);
    int8_t* lty = reinterpret_cast<int8_t*>(lsa + cell_cap);
    int32_t* ldel = reinterpret_cast<int32_t*>(lty + cell_cap);
    __shared__ int32_t ljs[kMaxCpmTypes * kMaxCpmTypes];
    if (c & 1)
        quad_pass<1>(a, c, sweep_off, qthr, lsa, lty, ljs, ldel);
    else
        quad_pass<0>(a, c, sweep_off, qthr, lsa, lty, ljs, ldel);
}

__global__ void __launch_bounds__(1024) k_cpm_pass_site(CpmArgs a, int c, int sweep_off,
                                                        int tab_lds_bytes, int cell_cap) {
    // dynamic LDS as k_cpm_pass_quad
    extern __shared__ __align__(16) uint8_t dyn[];
    uint32_t* qthr = reinterpret_cast<uint32_t*>(dyn);
    int32_t* lsa = reinterpret_cast<int32_t*>(dyn + tab_lds_bytes);
    int8_t* lty = reinterpret_cast<int8_t*>(lsa + cell_cap);
    int32_t* ldel = reinterpret_cast<int32_t*>(lty + cell_cap);
    __shared__ int32_t ljs[kMaxCpmTypes * kMaxCpmTypes];
    if (c & 1)
        site_pass<1>(a, c, sweep_off, qthr, lsa, lty, ljs, ldel);
    else
        site_pass<0>(a, c, sweep_off, qthr, lsa, lty, ljs, ldel);
}

// ------------------------------------------------------- two-phase attempts
// Most attempts end at once: the chosen neighbour holds the site's own id.
// A wave therefore works in two phases.  The first takes one Philox block of
// four attempts per lane, looks at nothing but the two ids, and queues the
// attempts that have to be decided (in LDS, in the wave's own segment, so
// that no barrier lies between); the second decides the queued ones, one per
// lane, so that no lane waits through a decision it does not have.  (One
// attempt per lane, decided in place, ran every wave that held one boundary
// site through the whole decision and computed each block four times.)
namespace {

// Queue entry: the attempt's accept prefix (bits 16..31), its place (up to 11 bits:
// four times the lane plus the word; where a pass is one round of up to 512 blocks,
// its within-colour index) and the chosen neighbour (range 1: 3 bits, range 2: 5).
template <int RANGE>
struct Entry {
    static constexpr int kShift = RANGE == 1 ? 3 : 5;
    static __device__ __forceinline__ uint32_t make(uint32_t word, uint32_t place, uint32_t jn) {
        return (word & 0xFFFF0000u) | (place << kShift) | jn;
    }
    static __device__ __forceinline__ int place(uint32_t e) { return (int)((e & 0xFFFFu) >> kShift); }
    static __device__ __forceinline__ int lane(uint32_t e) { return (int)(e >> (kShift + 2)) & 63; }
    static __device__ __forceinline__ int word(uint32_t e) { return (int)(e >> kShift) & 3; }
    static __device__ __forceinline__ uint32_t jn(uint32_t e) { return e & ((1u << kShift) - 1u); }
};

// Ids carry their cell's type, times eight, in the top byte: a type count is
// one shift-and-add, and ids compare as whole words.
__device__ __forceinline__ int id_of(uint32_t v) { return (int)(v & 0xFFFFFFu); }

// Adhesion change for all pairs (type of the present id, type of the copied
// one): d[t] = J[new][t] - J[old][t] per neighbour type, and the two diagonal
// terms J[new][new], J[old][old] of neighbours that hold the id itself.
struct PairTab {
    int4 d[16];
    int2 diag[16];
};

__device__ __forceinline__ void stage_pairs(const CpmArgs& a, const RepDev& R, PairTab* T, int tid) {
    if (tid >= 16) return;
    const int ts = tid >> 2, tt = tid & 3, nt = R.n_types;
    const int32_t* js = a.js + R.js_off;
    int v[4] = {0, 0, 0, 0};
    int2 dg = make_int2(0, 0);
    if (ts < nt && tt < nt) {
        for (int t = 0; t < nt; ++t) v[t] = js[tt * nt + t] - js[ts * nt + t];
        dg = make_int2(js[tt * nt + tt], js[ts * nt + ts]);
    }
    T->d[tid] = make_int4(v[0], v[1], v[2], v[3]);
    T->diag[tid] = dg;
}

// The decision of one attempt: old id s, copied id tg (packed with types),
// cnt the neighbours' type counts (a byte each), nt / ns how many neighbours
// hold tg / s; da / db the pass-start area minus target of tg and s (not used
// for the medium; R.small_areas is uniform).  Prefix r of W from the entry; the low half from the
// fallback block of k.
__device__ __forceinline__ bool cpm_accept(const CpmArgs& a, const RepDev& R, uint32_t s, uint32_t tg,
                                           uint32_t cnt, int nt, int ns, const PairTab* T, int da,
                                           int db, const uint32_t* thr, uint32_t r, uint32_t k,
                                           uint32_t p) {
    const int pi = (int)((s >> 27) * 4u + (tg >> 27));
    const int4 d = T->d[pi];
    const int2 dg = T->diag[pi];
    const int kadh = __mul24((int)(cnt & 0xFFu), d.x) + __mul24((int)((cnt >> 8) & 0xFFu), d.y) +
                     __mul24((int)((cnt >> 16) & 0xFFu), d.z) + __mul24((int)(cnt >> 24), d.w) -
                     __mul24(nt, dg.x) + __mul24(ns, dg.y);
    const bool ct = id_of(tg) != 0, cs = id_of(s) != 0;
    const int xa = ct ? da : 0, xb = cs ? db : 0;
    int64_t kk;
    if (R.small_areas)  // the area term fits 32 bits, lambda S always does
        kk = (int64_t)kadh + (int64_t)(int32_t)R.LS * (int64_t)(2 * (xa - xb) + ct + cs);
    else
        kk = (int64_t)kadh + R.LS * (2 * ((int64_t)xa - (int64_t)xb) + ct + cs);
    if (kk <= 0) return true;
    if (kk >= R.K0) return false;
    uint32_t hi = 0u, lo = 1u;  // T = 1 for K1 <= k < K0
    const bool tab = kk < (int64_t)R.K1;
    if (tab) hi = thr[kk - 1];
    if (r != hi) return r < hi;
    if (tab) lo = thr[R.tab_n + kk - 1];
    if (lo == 0u) return false;
    uint32_t f[4];
    philox4x32_10(k, p, R.rid, kTagFallback, a.key0, a.key1, f);
    return (f[0] & 0xFFFFu) < lo;
}

// The wave's queued attempts (act[u] per word u) into its segment, by the
// lanes' prefix counts; returns their number (uniform over the wave).
__device__ __forceinline__ int queue_put(uint32_t* queue, const bool (&act)[4],
                                         const uint32_t (&e)[4]) {
    int total = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint64_t m = __ballot(act[u]);
        if (act[u])
            queue[__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                            __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)total))] =
                e[u];
        total += __popcll(m);
    }
    // the other lanes of the wave read the entries
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return total;
}

// The neighbour's offset for neighbour j of a lattice of row stride st.
// Moore (range 1): the table holds offset + st + 1 for the eight neighbours,
// low and high bytes apart, so that two byte permutes look it up.
struct MooreTab {
    uint32_t lo0, lo1, hi0, hi1;
};
__device__ __forceinline__ MooreTab moore_tab(int st) {
    const int o[8] = {0, 1, 2, st, st + 2, 2 * st, 2 * st + 1, 2 * st + 2};
    MooreTab t = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        t.lo0 |= (uint32_t)(o[j] & 255) << (8 * j);
        t.hi0 |= (uint32_t)(o[j] >> 8) << (8 * j);
        t.lo1 |= (uint32_t)(o[j + 4] & 255) << (8 * j);
        t.hi1 |= (uint32_t)(o[j + 4] >> 8) << (8 * j);
    }
    return t;
}
__device__ __forceinline__ int moore_offset(const MooreTab& t, uint32_t word) {
    const uint32_t sel = (word & 7u) | 0x0C0C0C00u;
    return (int)(__builtin_amdgcn_perm(t.lo1, t.lo0, sel) |
                 (__builtin_amdgcn_perm(t.hi1, t.hi0, sel) << 8));
}
// 5x5 (range 2): neighbour j of 24 in row-major order without the centre
__device__ __forceinline__ int offset5(uint32_t j, int st) {
    const uint32_t jj = j < 12u ? j : j + 1u;
    const uint32_t dy = __umul24(jj, 13u) >> 6;  // jj / 5 for jj < 25
    return (int)(__umul24(dy, (uint32_t)st) + jj - __umul24(dy, 5u));
}

// exact quotient b / d for b < 2^16 from m = floor((2^32 - 1) / d) + 1; d > 1 (for
// 1, m wraps to 0), which the host sees to for the widths of a colour's rows
__device__ __forceinline__ int mdiv(int b, uint32_t m) { return (int)__umulhi((uint32_t)b, m); }
__device__ __forceinline__ uint32_t mdiv_of(int d) { return 0xFFFFFFFFu / (uint32_t)d + 1u; }

// The statistics of k_cpm_stats and k_cpm_area_energy from the LDS lattice
// (row stride st, the first site at o0): boundary bonds by type pair into
// lpair, the fixed-point energy into lH; sa + da is area minus target.
template <int RANGE>
__device__ __forceinline__ void cpm_lds_stats(const CpmArgs& a, const RepDev& R, const uint32_t* lids,
                                              int o0, int st, uint32_t mL, const int32_t* sa,
                                              const int32_t* da, int* lpair,
                                              unsigned long long* lH) {
    const int Lx = R.Lx, n = Lx * R.Ly, nt = R.n_types;
    const int32_t* js = a.js + R.js_off;
    long long H = 0;
    for (int it = (int)threadIdx.x; it < n; it += (int)blockDim.x) {
        const int y = mdiv(it, mL), x = it - y * Lx;
        const uint32_t* q = lids + o0 + y * st + x;
        const uint32_t s = q[0];
        constexpr int kN = RANGE == 2 ? 12 : 4;  // forward half of the neighbourhood
        const int dy[12] = {0, 1, 1, 1, 0, 1, 1, 2, 2, 2, 2, 2};
        const int dx[12] = {1, 0, 1, -1, 2, -2, 2, -2, -1, 0, 1, 2};
#pragma unroll
        for (int j = 0; j < kN; ++j) {
            const uint32_t m = q[dy[j] * st + dx[j]];
            if (m == s) continue;
            const int ts = (int)(s >> 27), tm = (int)(m >> 27);
            H += js[ts * nt + tm];
            if (j < 2) {  // von Neumann bonds
                const int p0 = min(ts, tm), p1 = max(ts, tm);
                atomicAdd(&lpair[p0 * nt - p0 * (p0 - 1) / 2 + (p1 - p0)], 1);
            }
        }
    }
    for (int i = 1 + (int)threadIdx.x; i <= R.q; i += (int)blockDim.x) {
        const long long d = (long long)(sa[i] + da[i]);
        H += R.LS * d * d;
    }
    for (int o = 32; o > 0; o >>= 1) H += __shfl_xor(H, o, 64);
    if ((threadIdx.x & 63) == 0) atomicAdd(lH, (unsigned long long)H);
}

}  // namespace

namespace {

// The four attempts of block b in pass p from their random words: queue
// entries e and the chosen neighbours' offsets off in the padded lattice,
// from the window's first id; place of the first.
template <int RANGE>
__device__ __forceinline__ void cpm_draw(const CpmArgs& a, const RepDev& R, const MooreTab& moore,
                                         int st, int b, int place, uint32_t p, uint32_t (&e)[4],
                                         uint32_t (&off)[4]) {
    uint32_t w[4];
    philox4x32_10((uint32_t)b, p, R.rid, kTagMain, a.key0, a.key1, w);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t k = 4u * (uint32_t)b + (uint32_t)u;
        uint32_t jn;
        if (RANGE == 1) {
            jn = w[u] & 7u;
            off[u] = (uint32_t)moore_offset(moore, jn);
        } else {
            // 24 neighbours: Lemire's multiply-shift of the low 16 bits,
            // redrawn from the fallback block on rejection
            const uint32_t l = __umul24(w[u] & 0xFFFFu, 24u);
            jn = l >> 16;
            if ((l & 0xFFFFu) < 16u) {
                uint32_t f[4];
                philox4x32_10(k, p, R.rid, kTagFallback, a.key0, a.key1, f);
                jn = (uint32_t)(((uint64_t)f[1] * 24u) >> 32);
            }
            off[u] = (uint32_t)offset5(jn, st);
        }
        e[u] = Entry<RANGE>::make(w[u], (uint32_t)(place + u), jn);
    }
}

}  // namespace

// All n_steps Monte Carlo steps of every replica in one launch: one workgroup
// per replica with its ids (with a halo of the neighbourhood's width, so that
// no neighbour wraps), areas, cell tables and thresholds in LDS, one barrier a
// pass.  A block's four sites are consecutive within-colour indices; ROWS (range 1,
// Lx % 8 == 0): all of one row; groups of eight blocks go round the waves, so that
// the cells' boundaries spread over them.  Areas minus targets rotate as in
// the streamed passes: pass P reads S[P & 1] + D[(P - 1) % 3] and adds its
// changes into D[P % 3] with LDS atomics, S and D of pass P + 1 are prepared
// on the side.  GEN (lattices of up to 512 blocks a pass): as many waves again
// draw the next pass's attempts into LDS and rotate the areas meanwhile, so
// that the deciding waves' chain holds only reads of ids and decisions;
// otherwise every wave draws its own.  re > 0: after step sw0 + st + 1 = j re
// of the call the statistics go to stats row j - 1.
// Bound by the chain of LDS reads and dependent instructions of a pass's few
// waves per SIMD: 256 replicas of 64 x 64 with 36 cells took 7.5 us a step
// with one attempt per lane decided in place, 6.7 with two phases around a
// barrier and a branch per site, 6.0 without those, 5.6 with the drawing
// waves.
template <int RANGE, bool GEN, bool ROWS>
__global__ void __launch_bounds__(1024) k_cpm_resident(CpmArgs a, int n_steps, int sw0, int re,
                                                       int tab_lds_bytes, int cell_cap,
                                                       int queue_words) {
    // dynamic LDS: [T hi | T lo] (tab_lds_bytes) | S[2], D[3] (int32 [cell_cap]
    // each) | queue (256 words per deciding wave) | GEN: drawn entries (uint4)
    // and offsets (four 16-bit) per deciding lane, two passes | ids with halo
    extern __shared__ __align__(16) uint8_t dyn[];
    __shared__ PairTab pairs;
    __shared__ int lpair[10];
    __shared__ unsigned long long lH;
    constexpr int ncol = RANGE == 2 ? 9 : 4, P = RANGE == 2 ? 3 : 2;  // colours, period
    constexpr int h = RANGE;                                         // halo
    uint32_t* qthr = reinterpret_cast<uint32_t*>(dyn);
    int32_t* lS = reinterpret_cast<int32_t*>(dyn + tab_lds_bytes);
    int32_t* lD = lS + 2 * cell_cap;
    const RepDev R = a.reps[blockIdx.x];
    const int Lx = R.Lx, Ly = R.Ly, st = Lx + 2 * h;
    const int ncell = R.q + 1, nthr = (int)blockDim.x, tid = (int)threadIdx.x;
    const int ndec = GEN ? nthr >> 1 : nthr;  // deciding lanes
    const bool gen = GEN && tid >= ndec;      // uniform over a wave
    const int dt = gen ? tid - ndec : tid;    // the lane's place among its kind
    const int wave = dt >> 6, lane = tid & 63, nw = ndec >> 6;
    uint32_t* queue0 = reinterpret_cast<uint32_t*>(lD + 3 * cell_cap);
    uint32_t* queue = queue0 + 256 * wave;
    uint4* gE = reinterpret_cast<uint4*>(queue0 + queue_words);
    uint2* gO = reinterpret_cast<uint2*>(gE + 2 * ndec);
    uint32_t* lids = GEN ? reinterpret_cast<uint32_t*>(gO + 2 * ndec) : queue0 + queue_words;
    uint32_t* gids = reinterpret_cast<uint32_t*>(a.lat + R.lat_off);
    int32_t* garea = a.area + R.cell_off;
    const int32_t* gA = a.target + R.cell_off;
    const int8_t* ty = a.ctype + R.cell_off;
    for (int i = tid; i < 2 * R.tab_n; i += nthr) qthr[i] = a.tab[R.tab_off + i];
    stage_pairs(a, R, &pairs, tid);
    const uint64_t t0 = *a.t_base;
    // rotating areas for the first pass P0 = ncol t0
    int sp = (int)((ncol * t0) & 1u), dp = (int)((ncol * t0) % 3u);  // P & 1, P % 3
    for (int i = tid; i < ncell; i += nthr) {
        lS[sp * cell_cap + i] = garea[i] - gA[i];
        lD[i] = lD[cell_cap + i] = lD[2 * cell_cap + i] = 0;
    }
    for (int i = tid; i < st * (Ly + 2 * h); i += nthr) {
        const int y = i / st, x = i - y * st;
        const uint32_t v = gids[wrapc(y - h, Ly) * Lx + wrapc(x - h, Lx)];
        lids[i] = v | ((uint32_t)ty[v] << 27);
    }
    const int Wc = Lx / P, n_sites = (Ly / P) * Wc;  // sites per colour row and colour
    const int n_blk = (n_sites + 3) >> 2;
    const uint32_t mW = mdiv_of(Wc), mL = mdiv_of(Lx);
    const MooreTab moore = moore_tab(st);
    // block of the lane in round j: eight consecutive ones per eight lanes,
    // the groups of eight dealt out to the waves
    const auto block_of = [=](int l) { return ((l >> 3) * nw + wave) * 8 + (l & 7); };
    const int b0 = block_of(lane);
    uint32_t e[4], off[4];
    const auto put = [&](int buf) {
        gE[buf * ndec + dt] = make_uint4(e[0], e[1], e[2], e[3]);
        gO[buf * ndec + dt] = make_uint2(off[0] | (off[1] << 16), off[2] | (off[3] << 16));
    };
    if (gen) {
        cpm_draw<RANGE>(a, R, moore, st, b0, 4 * b0, (uint32_t)(ncol * t0), e, off);
        put(sp);
    }
    __syncthreads();
    int next = re > 0 ? (sw0 / re + 1) * re - sw0 : 0;  // steps to the next recorded one
    for (int step = 0; step < n_steps; ++step) {
        for (int c = 0; c < ncol; ++c) {
            const uint32_t p = (uint32_t)(ncol * (t0 + (uint64_t)step) + (uint64_t)c);
            const int cy = c / P, cx = c - P * cy;
            const int dq = dp == 0 ? 2 : dp - 1, dn = dp == 2 ? 0 : dp + 1;
            const int32_t* S0 = lS + sp * cell_cap;
            const int32_t* D0 = lD + dq * cell_cap;
            int32_t* D1 = lD + dp * cell_cap;
            if (!GEN || gen) {
                for (int i = GEN ? dt : tid; i < ncell; i += ndec) {
                    lS[(sp ^ 1) * cell_cap + i] = S0[i] + D0[i];
                    lD[dn * cell_cap + i] = 0;
                }
            }
            if (gen) {
                cpm_draw<RANGE>(a, R, moore, st, b0, 4 * b0, p + 1u, e, off);
                put(sp ^ 1);
            }
            // offset of the colour's site (0, 0), one row and column up-left
            // of it for the neighbour tables
            const int oc = (cy + h) * st + cx + h, on = oc - h * st - h;
            // every lane takes part (ballots); blocks past the end queue nothing
            for (int g = 0; g < n_blk && !gen; g += ndec) {
                const int b = g + b0;
                if (GEN) {
                    const uint4 ev = gE[sp * ndec + dt];
                    const uint2 ov = gO[sp * ndec + dt];
                    e[0] = ev.x; e[1] = ev.y; e[2] = ev.z; e[3] = ev.w;
                    off[0] = ov.x & 0xFFFFu; off[1] = ov.x >> 16;
                    off[2] = ov.y & 0xFFFFu; off[3] = ov.y >> 16;
                } else {
                    cpm_draw<RANGE>(a, R, moore, st, b, 4 * lane, p, e, off);
                }
                bool act[4];
                int r = mdiv(4 * b, mW), i = 4 * b - (int)__umul24((uint32_t)r, (uint32_t)Wc);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bool in = ROWS ? b < n_blk : 4 * b + u < n_sites;
                    const int o = in ? P * ((int)__umul24((uint32_t)r, (uint32_t)st) + i) : 0;
                    // (no branch around the reads: all of the block's together)
                    act[u] = (lids[oc + o] != lids[on + o + (int)off[u]]) & in;
                    ++i;  // the block's next site
                    if (!ROWS && i == Wc) {
                        i = 0;
                        ++r;
                    }
                }
                const int cnt_q = queue_put(queue, act, e);
                for (int q = lane; q < cnt_q; q += 64) {
                    const uint32_t v = queue[q], jn = Entry<RANGE>::jn(v);
                    const uint32_t k = (uint32_t)(
                        GEN ? Entry<RANGE>::place(v)
                            : 4 * (g + block_of(Entry<RANGE>::lane(v))) + Entry<RANGE>::word(v));
                    const int r2 = mdiv((int)k, mW);
                    const int i2 = (int)k - (int)__umul24((uint32_t)r2, (uint32_t)Wc);
                    const int o = P * ((int)__umul24((uint32_t)r2, (uint32_t)st) + i2);
                    const uint32_t* nb = lids + on + o;  // the window's first id
                    const uint32_t s = nb[h * st + h];
                    const uint32_t tg =
                        nb[RANGE == 1 ? moore_offset(moore, jn) : offset5(jn, st)];
                    uint32_t cnt = 0u;
                    int nt = 0, ns = 0;
#pragma unroll
                    for (int dy = 0; dy <= 2 * h; ++dy)
#pragma unroll
                        for (int dx = 0; dx <= 2 * h; ++dx) {
                            if (dy == h && dx == h) continue;  // the site itself
                            const uint32_t m = nb[dy * st + dx];
                            cnt += 1u << (m >> 24);
                            nt += m == tg;
                            ns += m == s;
                        }
                    const int it = id_of(tg), is = id_of(s);
                    if (cpm_accept(a, R, s, tg, cnt, nt, ns, &pairs, S0[it] + D0[it],
                                   S0[is] + D0[is], qthr, v >> 16, k, p)) {
                        const int y = P * r2 + cy, x = P * i2 + cx;
                        uint32_t* d = lids + oc + o;
                        *d = tg;
                        // the halo's copies
                        const int xe = x < h ? Lx : (x >= Lx - h ? -Lx : 0);
                        const int ye = (y < h ? Ly : (y >= Ly - h ? -Ly : 0)) * st;
                        if (xe != 0) d[xe] = tg;
                        if (ye != 0) d[ye] = tg;
                        if (xe != 0 && ye != 0) d[xe + ye] = tg;
                        atomicAdd(&D1[it], 1);
                        atomicAdd(&D1[is], -1);
                    }
                }
                // the queue is read before the next round's entries
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            sp ^= 1;
            dp = dn;
            __syncthreads();
        }
        if (re > 0 && step + 1 == next) {
            next += re;
            if (tid < 10) lpair[tid] = 0;
            if (tid == 0) lH = 0ull;
            __syncthreads();
            cpm_lds_stats<RANGE>(a, R, lids, h * st + h, st, mL, lS + sp * cell_cap,
                                 lD + (dp == 0 ? 2 : dp - 1) * cell_cap, lpair, &lH);
            __syncthreads();
            int32_t* row = a.stats + ((size_t)((sw0 + step + 1) / re - 1) * a.R + blockIdx.x) * a.width;
            for (int i = tid; i < a.width; i += nthr)
                row[i] = i < 10 ? lpair[i]
                                : (i == 10 ? (int32_t)(uint32_t)lH
                                           : (i == 11 ? (int32_t)(uint32_t)(lH >> 32) : 0));
        }
    }
    for (int i = tid; i < Lx * Ly; i += nthr) {
        const int y = i / Lx, x = i - y * Lx;
        gids[i] = (uint32_t)id_of(lids[(y + h) * st + x + h]);
    }
    for (int i = tid; i < ncell; i += nthr) {
        const int v = lS[sp * cell_cap + i] + lD[(dp == 0 ? 2 : dp - 1) * cell_cap + i] + gA[i];
        garea[i] = v;
        a.snap[R.cell_off + i] = v;
    }
}

// ------------------------------------------------------ streamed, two phases
// One colour pass over tiles of rows x columns (range 1, every Lx % 8 == 0):
// the tile's ids with a halo come into LDS in 16-byte loads, together with the
// thresholds and the cells' tables -- one round of global loads, none of them
// waiting for another but for the tile's record -- and the attempts run on the
// LDS ids in the two phases of the resident kernel.  Accepted ids go straight
// to the lattice; area changes gather in LDS and go to the pass's change
// buffer as one atomic per touched cell (without TAB: types and areas are read from
// memory and changed there, by the decided attempts alone).  Bound by latencies: launch, the tile
// record, the loads, the chain of LDS reads, the stores.  8 x 512^2, 1000
// cells: 9.0 us a pass with one attempt per lane on a register window,
// 6.5 now.
template <bool TAB>
__global__ void __launch_bounds__(512) k_cpm_pass_tile(CpmArgs a, const CpmTile* tiles, int c,
                                                       int sweep_off, int tab_lds_bytes,
                                                       int cell_cap) {
    // dynamic LDS (cell_cap 0 without TAB): [T hi | T lo] (tab_lds_bytes) | snap - A, area changes (int32
    // [cell_cap] each) | 8 x type (int8 [cell_cap]) | queue (256 words per wave)
    // | ids: (rows + 2) x (cols + 8), four halo columns on either side
    extern __shared__ __align__(16) uint8_t dyn[];
    __shared__ PairTab pairs;
    const CpmTile& T = tiles[blockIdx.x];
    const RepDev R = T.R;
    const int tid = (int)threadIdx.x, nthr = (int)blockDim.x, lane = tid & 63;
    uint32_t* qthr = reinterpret_cast<uint32_t*>(dyn);
    int32_t* lsa = reinterpret_cast<int32_t*>(dyn + tab_lds_bytes);
    int32_t* ldel = lsa + cell_cap;
    uint8_t* lty = reinterpret_cast<uint8_t*>(ldel + cell_cap);
    uint32_t* queue0 = reinterpret_cast<uint32_t*>(lty + cell_cap);
    uint32_t* queue = queue0 + 256 * (tid >> 6);
    uint32_t* lids = queue0 + 4 * nthr;
    const int Lx = R.Lx, Ly = R.Ly, y0 = T.y0, x0 = T.x0, rows = T.rows, cols = T.cols;
    const int st = cols + 8, cw = st >> 2, nch = (rows + 2) * cw;  // 16-byte chunks
    int32_t* gids = a.lat + R.lat_off;
    const uint64_t P = 4 * (*a.t_base + (uint64_t)sweep_off) + (uint64_t)c;
    const uint32_t p = (uint32_t)P;
    const PassAreas pa = pass_areas(a, P, R.cell_off);
    const int ncell = R.q + 1, ntab = 2 * R.tab_n;
    const uint32_t mC = mdiv_of(cw);
    // every thread's first loads of each kind before any is used
    constexpr int kU = 5;
    int4 v[kU];
    const auto chunk = [&](int i) {
        const int r = mdiv(i, mC), j = i - r * cw;
        int gx = x0 - 4 + 4 * j;
        gx = gx < 0 ? gx + Lx : (gx >= Lx ? gx - Lx : gx);
        return *reinterpret_cast<const int4*>(gids + (size_t)wrapc(y0 + r - 1, Ly) * Lx + gx);
    };
#pragma unroll
    for (int u = 0; u < kU; ++u)
        if (tid + u * nthr < nch) v[u] = chunk(tid + u * nthr);
    constexpr int kC = 2;
    int32_t sv[kC], av[kC];
    uint8_t tv[kC];
    const int nst = TAB ? ncell : 0;  // cells staged
    const int32_t* gA = a.target + R.cell_off;
    const int8_t* gty = a.ctype + R.cell_off;
#pragma unroll
    for (int u = 0; u < kC; ++u) {
        const int i = tid + u * nthr;
        if (i < nst) {
            sv[u] = pa.s_rd[i] + pa.d_rd[i];
            av[u] = gA[i];
            tv[u] = (uint8_t)gty[i];
        }
    }
    for (int i = tid; i < ntab; i += nthr) qthr[i] = a.tab[R.tab_off + i];
    stage_pairs(a, R, &pairs, tid);
#pragma unroll
    for (int u = 0; u < kC; ++u) {
        const int i = tid + u * nthr;
        if (i < nst) {
            lsa[i] = sv[u] - av[u];
            lty[i] = (uint8_t)(8 * tv[u]);
            ldel[i] = 0;
        }
    }
    for (int i = tid + kC * nthr; i < nst; i += nthr) {
        lsa[i] = pa.s_rd[i] + pa.d_rd[i] - gA[i];
        lty[i] = (uint8_t)(8 * gty[i]);
        ldel[i] = 0;
    }
    const auto type8 = [&](uint32_t m) { return TAB ? (uint32_t)lty[m] : 8u * (uint32_t)gty[m]; };
    const auto over = [&](uint32_t m) {  // pass-start area minus target
        return TAB ? lsa[m] : pa.s_rd[m] + pa.d_rd[m] - gA[m];
    };
#pragma unroll
    for (int u = 0; u < kU; ++u)
        if (tid + u * nthr < nch) reinterpret_cast<int4*>(lids)[tid + u * nthr] = v[u];
    for (int i = tid + kU * nthr; i < nch; i += nthr) reinterpret_cast<int4*>(lids)[i] = chunk(i);
    pass_rotate(a, P);
    __syncthreads();
    const int cy = c >> 1, cx = c & 1;
    const int Gt = cols >> 3, G = Lx >> 3, nq = (rows >> 1) * Gt;  // quads of the tile's colour
    const uint32_t mG = Gt > 1 ? mdiv_of(Gt) : 0u;
    const auto qrow = [&](int b) { return Gt > 1 ? mdiv(b, mG) : b; };
    const MooreTab moore = moore_tab(st);
    const int oc = (cy + 1) * st + cx + 4, on = oc - st - 1;
    // every lane takes part (ballots); quads past the end queue nothing
    for (int g = 0; g < nq; g += nthr) {
        const int b = g + tid;
        const bool in = b < nq;
        const int r = in ? qrow(b) : 0, j = in ? b - (int)__umul24((uint32_t)r, (uint32_t)Gt) : 0;
        const uint32_t kq = (uint32_t)((y0 >> 1) + r) * (uint32_t)G + (uint32_t)((x0 >> 3) + j);
        uint32_t w[4];
        philox4x32_10(kq, p, R.rid, kTagMain, a.key0, a.key1, w);
        const int o = 2 * (int)__umul24((uint32_t)r, (uint32_t)st) + 8 * j;
        bool act[4];
        uint32_t e[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            // (no branch around the reads: all of the quad's together)
            act[u] = (lids[oc + o + 2 * u] !=
                      lids[on + o + 2 * u + moore_offset(moore, w[u])]) & in;
            e[u] = Entry<1>::make(w[u], (uint32_t)(4 * lane + u), w[u] & 7u);
        }
        const int cnt_q = queue_put(queue, act, e);
        for (int q = lane; q < cnt_q; q += 64) {
            const uint32_t ev = queue[q], jn = Entry<1>::jn(ev);
            const uint32_t kl = (uint32_t)Entry<1>::word(ev);
            const int b2 = g + (tid & ~63) + Entry<1>::lane(ev), r2 = qrow(b2);
            const int j2 = b2 - (int)__umul24((uint32_t)r2, (uint32_t)Gt);
            const int o2 = 2 * (int)__umul24((uint32_t)r2, (uint32_t)st) + 8 * j2 + 2 * (int)kl;
            const uint32_t* nb = lids + on + o2;
            const uint32_t s = nb[st + 1], tg = nb[moore_offset(moore, jn)];
            uint32_t cnt = 0u;
            int nt = 0, ns = 0;
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) {
                    if (dy == 1 && dx == 1) continue;
                    const uint32_t m = nb[dy * st + dx];
                    cnt += 1u << type8(m);
                    nt += m == tg;
                    ns += m == s;
                }
            const uint32_t k = 4u * ((uint32_t)((y0 >> 1) + r2) * (uint32_t)G +
                                     (uint32_t)((x0 >> 3) + j2)) + kl;
            if (cpm_accept(a, R, s | (type8(s) << 24), tg | (type8(tg) << 24), cnt, nt, ns, &pairs,
                           over(tg), over(s), qthr, ev >> 16, k, p)) {
                gids[(size_t)(y0 + 2 * r2 + cy) * Lx + x0 + 8 * j2 + 2 * (int)kl + cx] = (int)tg;
                atomicAdd(TAB ? &ldel[tg] : &pa.d_wr[tg], 1);
                atomicAdd(TAB ? &ldel[s] : &pa.d_wr[s], -1);
            }
        }
        // the queue is read before the next round's entries
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if (!TAB) return;
    __syncthreads();
    for (int i = tid; i < ncell; i += nthr) {
        const int d = ldel[i];
        if (d != 0) atomicAdd(&pa.d_wr[i], d);
    }
}

// The same pass over bands of whole rows, for every other lattice: range 2 (5x5,
// nine colours), and range 1 where Lx is not a multiple of 8.  T.rows (a multiple
// of the colouring's period) by T.cols = Lx; the ids come in dword by dword, a
// block's four sites may run on into the band's next row, and blocks at the band's
// ends belong to both bands, each deciding its own sites.  Bound as above; with two
// or more bands a compute unit by the staging of ids (about 12 dwords a lane).
// Without TAB the cells' tables stay in global memory, for the decided attempts alone.
// Range 2, 3 x 378^2, 364 cells: 7.1 us a pass with one attempt per lane deciding
// in place, 5.9 now; 8 x 510^2, 648 cells: 14.4 and 9.2; range 1, 430^2, 450 cells:
// 12.1 and 6.1; 8 x 510^2: 16.0 and 8.4.  With range 2 a lattice all of one cell is
// known by that cell's area and ends before its draws (216^2: 3.2 us, in place 3.1,
// without that 4.2; it costs the others 0.1).
template <int RANGE, bool TAB>
__global__ void __launch_bounds__(512) k_cpm_pass_band(CpmArgs a, const CpmTile* tiles, int c,
                                                       int sweep_off, int tab_lds_bytes,
                                                       int cell_cap) {
    // dynamic LDS as above, cell_cap 0 without TAB; ids: (rows + 2 h) x (Lx + 2 h),
    // h = RANGE
    extern __shared__ __align__(16) uint8_t dyn[];
    __shared__ PairTab pairs;
    constexpr int ncol = RANGE == 2 ? 9 : 4, P = RANGE == 2 ? 3 : 2, h = RANGE;
    const CpmTile& T = tiles[blockIdx.x];
    const RepDev R = T.R;
    const int tid = (int)threadIdx.x, nthr = (int)blockDim.x, lane = tid & 63;
    uint32_t* qthr = reinterpret_cast<uint32_t*>(dyn);
    int32_t* lsa = reinterpret_cast<int32_t*>(dyn + tab_lds_bytes);
    int32_t* ldel = lsa + cell_cap;
    uint8_t* lty = reinterpret_cast<uint8_t*>(ldel + cell_cap);
    uint32_t* queue0 = reinterpret_cast<uint32_t*>(lty + cell_cap);
    uint32_t* queue = queue0 + 256 * (tid >> 6);
    uint32_t* lids = queue0 + 4 * nthr;
    const int Lx = R.Lx, Ly = R.Ly, y0 = T.y0, rows = T.rows;
    const int st = Lx + 2 * h, nd = (rows + 2 * h) * st;
    int32_t* gids = a.lat + R.lat_off;
    const uint64_t PP = (uint64_t)ncol * (*a.t_base + (uint64_t)sweep_off) + (uint64_t)c;
    const uint32_t p = (uint32_t)PP;
    const PassAreas pa = pass_areas(a, PP, R.cell_off);
    const int ncell = R.q + 1, ntab = 2 * R.tab_n;
    const uint32_t mS = mdiv_of(st);
    // every thread's first loads of each kind before any is used
    constexpr int kU = 12;
    int32_t v[kU];
    const auto load = [&](int i) {
        const int r = mdiv(i, mS);
        return gids[(size_t)wrapc(y0 + r - h, Ly) * Lx + wrapc(i - r * st - h, Lx)];
    };
    const int32_t id0 = RANGE == 2 ? gids[(size_t)y0 * Lx] : 0;
#pragma unroll
    for (int u = 0; u < kU; ++u)
        if (tid + u * nthr < nd) v[u] = load(tid + u * nthr);
    const int32_t area0 = RANGE == 2 ? pa.s_rd[id0] + pa.d_rd[id0] : 0;
    constexpr int kC = 2;
    int32_t sv[kC], av[kC];
    uint8_t tv[kC];
    const int nst = TAB ? ncell : 0;  // cells staged
    const int32_t* gA = a.target + R.cell_off;
    const int8_t* gty = a.ctype + R.cell_off;
#pragma unroll
    for (int u = 0; u < kC; ++u) {
        const int i = tid + u * nthr;
        if (i < nst) {
            sv[u] = pa.s_rd[i] + pa.d_rd[i];
            av[u] = gA[i];
            tv[u] = (uint8_t)gty[i];
        }
    }
    for (int i = tid; i < ntab; i += nthr) qthr[i] = a.tab[R.tab_off + i];
    stage_pairs(a, R, &pairs, tid);
#pragma unroll
    for (int u = 0; u < kC; ++u) {
        const int i = tid + u * nthr;
        if (i < nst) {
            lsa[i] = sv[u] - av[u];
            lty[i] = (uint8_t)(8 * tv[u]);
            ldel[i] = 0;
        }
    }
    for (int i = tid + kC * nthr; i < nst; i += nthr) {
        lsa[i] = pa.s_rd[i] + pa.d_rd[i] - gA[i];
        lty[i] = (uint8_t)(8 * gty[i]);
        ldel[i] = 0;
    }
    const auto type8 = [&](uint32_t m) { return TAB ? (uint32_t)lty[m] : 8u * (uint32_t)gty[m]; };
    const auto over = [&](uint32_t m) {  // pass-start area minus target
        return TAB ? lsa[m] : pa.s_rd[m] + pa.d_rd[m] - gA[m];
    };
#pragma unroll
    for (int u = 0; u < kU; ++u)
        if (tid + u * nthr < nd) lids[tid + u * nthr] = (uint32_t)v[u];
    for (int i = tid + kU * nthr; i < nd; i += nthr) lids[i] = (uint32_t)load(i);
    pass_rotate(a, PP);
    __syncthreads();
    // a lattice all of one cell has nothing to decide
    if (RANGE == 2 && __builtin_amdgcn_readfirstlane(area0) == Lx * Ly) return;
    const int cy = c / P, cx = c - P * cy;
    const int Wc = Lx / P, k0 = y0 / P * Wc, n = rows / P * Wc;  // the band's sites k0 .. k0 + n - 1
    const int blk0 = k0 >> 2, n_blk = ((k0 + n + 3) >> 2) - blk0;
    const uint32_t mW = mdiv_of(Wc);
    const MooreTab moore = moore_tab(st);
    const int oc = (cy + h) * st + cx + h, on = oc - h * st - h;
    // every lane takes part (ballots); sites outside the band queue nothing
    for (int g = 0; g < n_blk; g += nthr) {
        const int b = blk0 + g + tid;
        uint32_t e[4], off[4];
        cpm_draw<RANGE>(a, R, moore, st, b, 4 * lane, p, e, off);
        const int f = 4 * b - k0, f0 = max(f, 0);  // first site within the band
        int r = mdiv(f0, mW), i = f0 - r * Wc;
        bool act[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool in = f + u >= 0 && f + u < n;
            const int o = in ? P * ((int)__umul24((uint32_t)r, (uint32_t)st) + i) : 0;
            // (no branch around the reads: all of the block's together)
            act[u] = (lids[oc + o] != lids[on + o + (int)off[u]]) & in;
            if (f + u >= 0 && ++i == Wc) {
                i = 0;
                ++r;
            }
        }
        const int cnt_q = queue_put(queue, act, e);
        for (int q = lane; q < cnt_q; q += 64) {
            const uint32_t ev = queue[q], jn = Entry<RANGE>::jn(ev);
            const int k = 4 * (blk0 + g + (tid & ~63) + Entry<RANGE>::lane(ev)) + Entry<RANGE>::word(ev);
            const int r2 = mdiv(k - k0, mW), i2 = k - k0 - (int)__umul24((uint32_t)r2, (uint32_t)Wc);
            const uint32_t* nb = lids + on + P * ((int)__umul24((uint32_t)r2, (uint32_t)st) + i2);
            const uint32_t s = nb[h * st + h];
            const uint32_t tg = nb[RANGE == 1 ? moore_offset(moore, jn) : offset5(jn, st)];
            uint32_t cnt = 0u;
            int nt = 0, ns = 0;
#pragma unroll
            for (int dy = 0; dy <= 2 * h; ++dy)
#pragma unroll
                for (int dx = 0; dx <= 2 * h; ++dx) {
                    if (dy == h && dx == h) continue;  // the site itself
                    const uint32_t m = nb[dy * st + dx];
                    cnt += 1u << type8(m);
                    nt += m == tg;
                    ns += m == s;
                }
            if (cpm_accept(a, R, s | (type8(s) << 24), tg | (type8(tg) << 24), cnt, nt, ns, &pairs,
                           over(tg), over(s), qthr, ev >> 16, (uint32_t)k, p)) {
                gids[(size_t)(y0 + P * r2 + cy) * Lx + P * i2 + cx] = (int)tg;
                atomicAdd(TAB ? &ldel[tg] : &pa.d_wr[tg], 1);
                atomicAdd(TAB ? &ldel[s] : &pa.d_wr[s], -1);
            }
        }
        // the queue is read before the next round's entries
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if (!TAB) return;
    __syncthreads();
    for (int i = tid; i < ncell; i += nthr) {
        const int d = ldel[i];
        if (d != 0) atomicAdd(&pa.d_wr[i], d);
    }
}

size_t cpm_band_lds_bytes(int range, int tab_lds_bytes, int cell_cap, int threads, int rows,
                          int Lx) {
    return (size_t)tab_lds_bytes + (size_t)9 * cell_cap + (size_t)16 * threads +
           (size_t)4 * (rows + 2 * range) * (Lx + 2 * range);
}

namespace {
const void* band_fn(int range, bool tab) {
    if (range == 2) return (const void*)k_cpm_pass_band<2, false>;
    return tab ? (const void*)k_cpm_pass_band<1, true> : (const void*)k_cpm_pass_band<1, false>;
}
}  // namespace

hipError_t cpm_band_reserve_lds(int range, int cell_cap, size_t lds_bytes) {
    return hipFuncSetAttribute(band_fn(range, cell_cap > 0),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
}

hipError_t launch_cpm_pass_band(const CpmArgs& a, const CpmTile* tiles, int n_tiles, int c,
                                int sweep_off, int threads, int tab_lds_bytes, int cell_cap,
                                size_t lds_bytes, hipStream_t s) {
    CpmArgs b = a;
    void* args[] = {&b, &tiles, &c, &sweep_off, &tab_lds_bytes, &cell_cap};
    return hipLaunchKernel(band_fn(a.range, cell_cap > 0), dim3(n_tiles), dim3(threads), args,
                           lds_bytes, s);
}

size_t cpm_tile_lds_bytes(int tab_lds_bytes, int cell_cap, int threads, int rows, int cols) {
    return (size_t)tab_lds_bytes + (size_t)9 * cell_cap + (size_t)16 * threads +
           (size_t)4 * (rows + 2) * (cols + 8);
}

hipError_t cpm_tile_reserve_lds(int cell_cap, size_t lds_bytes) {
    return hipFuncSetAttribute(cell_cap > 0 ? (const void*)k_cpm_pass_tile<true>
                                            : (const void*)k_cpm_pass_tile<false>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
}

hipError_t launch_cpm_pass_tile(const CpmArgs& a, const CpmTile* tiles, int n_tiles, int c,
                                int sweep_off, int threads, int tab_lds_bytes, int cell_cap,
                                size_t lds_bytes, hipStream_t s) {
    if (cell_cap > 0)
        hipLaunchKernelGGL(k_cpm_pass_tile<true>, dim3(n_tiles), dim3(threads), lds_bytes, s, a,
                           tiles, c, sweep_off, tab_lds_bytes, cell_cap);
    else
        hipLaunchKernelGGL(k_cpm_pass_tile<false>, dim3(n_tiles), dim3(threads), lds_bytes, s, a,
                           tiles, c, sweep_off, tab_lds_bytes, 0);
    return hipGetLastError();
}

// ------------------------------------------- tiled persistent streamed passes
// All 4 G colour passes of G unrecorded Monte Carlo steps in one launch for
// lattices too large for one workgroup's LDS (range 1, Lx % 8 == 0): every
// replica is cut into TH x TW tiles, one workgroup per tile for the whole
// launch, its ids (with a one-cell halo) in LDS.  A pass: the tile's sites
// of the colour attempt their copies on the LDS ids (the decision of the
// streamed passes, cpm_decide), the tile's border cells go to the global
// lattice and its area changes to the pass's change buffer; then the
// replica's workgroups meet at a barrier (a counter per replica, agent-scope
// release / acquire), after which each reads its halo ring, which the
// neighbouring tiles wrote, and stages the next pass's snapshot.  Snapshots
// rotate as in the streamed passes (S[P & 1] + D[(P-1) % 3], the side work of
// pass P spread over the replica's tiles).  Every tile workgroup of the
// launch must be resident at once (the host sizes the grid within the chip's
// occupancy); a barrier wait beyond its bound (about two seconds) raises
// *abort and every waiting workgroup leaves, so a launch always ends.
constexpr uint32_t kCpmSpinCap = 1u << 25;

__device__ __forceinline__ void cpm_wait_stores() { __builtin_amdgcn_s_waitcnt(0x0F70); }

__device__ int cpm_tile_barrier(uint32_t* bar, uint32_t need, uint32_t* abort_flag) {
    // release: the fence writes the L2 back (border ids, snapshot and change
    // buffers reach memory for the other XCDs), the explicit vmcnt(0) waits
    // for that write-back to finish, and only then is the arrival counted.
    // (A release add alone compiles to the write-back directly followed by
    // the add, with no wait between them, when the workgroup's stores were
    // already waited for, so a workgroup on another XCD could pass the
    // barrier and read memory the write-back had not reached.)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    cpm_wait_stores();
    __hip_atomic_fetch_add(bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (uint32_t spin = 0;; ++spin) {
        if (__hip_atomic_load(bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= need) break;
        if (__hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) return 0;
        if (spin >= kCpmSpinCap) {
            __hip_atomic_store(abort_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return 0;
        }
        __builtin_amdgcn_s_sleep(2);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return 1;
}

__global__ void __launch_bounds__(256) k_cpm_tiled(CpmArgs a, int n_steps, int TH, int TW,
                                                   int tab_lds_bytes, int cell_cap,
                                                   uint32_t* bar, uint32_t* abort_flag) {
    // dynamic LDS: [T hi | T lo] (tab_lds_bytes) | snap - A (int32 [cell_cap]) |
    // type (int8 [cell_cap], padded to 16) | ids with halo (int32 [TH + 2][TW + 2])
    extern __shared__ __align__(16) uint8_t dyn[];
    uint32_t* qthr = reinterpret_cast<uint32_t*>(dyn);
    int32_t* lsa = reinterpret_cast<int32_t*>(dyn + tab_lds_bytes);
    int8_t* lty = reinterpret_cast<int8_t*>(lsa + cell_cap);
    int32_t* tile = reinterpret_cast<int32_t*>(lty + ((cell_cap + 15) & ~15));
    __shared__ int32_t ljs[kMaxCpmTypes * kMaxCpmTypes];
    __shared__ int go;
    // block b: replica b % R, tile b / R (with R a multiple of 8 a replica's
    // tiles share one XCD)
    const int r = (int)blockIdx.x % a.R, tix = (int)blockIdx.x / a.R;
    const RepDev R = a.reps[r];
    const int Lx = R.Lx, Ly = R.Ly, ntx = Lx / TW, n_tiles = ntx * (Ly / TH);
    const int y0 = (tix / ntx) * TH, x0 = (tix % ntx) * TW;
    const int ts = TW + 2, nthr = (int)blockDim.x, tid = (int)threadIdx.x;
    const int ncell = R.q + 1;
    int32_t* gids = a.lat + R.lat_off;
    const int32_t* A = a.target + R.cell_off;
    for (int i = tid; i < 2 * R.tab_n; i += nthr) qthr[i] = a.tab[R.tab_off + i];
    for (int i = tid; i < R.n_types * R.n_types; i += nthr) ljs[i] = a.js[R.js_off + i];
    for (int i = tid; i < ncell; i += nthr) lty[i] = a.ctype[R.cell_off + i];
    // the tile with its halo (periodic)
    for (int i = tid; i < (TH + 2) * ts; i += nthr) {
        const int ly = i / ts, lx = i - ly * ts;
        const int gy = wrapc(y0 + ly - 1, Ly), gx = wrapc(x0 + lx - 1, Lx);
        tile[i] = gids[gy * Lx + gx];
    }
    const uint64_t t0 = *a.t_base;
    const int Q = Lx >> 3;                 // quads per global row
    const int nq = (TH >> 1) * (TW >> 3);  // quads of one colour in the tile
    // this tile's share of the replica's cells for the side work
    const int per = (ncell + n_tiles - 1) / n_tiles;
    const int c0 = tix * per, c1 = min(ncell, c0 + per);
    for (int sw = 0; sw < n_steps; ++sw) {
        for (int c = 0; c < 4; ++c) {
            const uint32_t j = (uint32_t)(4 * sw + c);
            const uint64_t P = 4 * (t0 + (uint64_t)sw) + (uint64_t)c;
            const uint32_t p = (uint32_t)P;
            const PassAreas pa = pass_areas(a, P, R.cell_off);
            if (j > 0) {
                // the halo ring, written by the neighbouring tiles' last pass
                const int ring = 2 * ts + 2 * TH;
                for (int i = tid; i < ring; i += nthr) {
                    int ly, lx;
                    if (i < ts) {
                        ly = 0;
                        lx = i;
                    } else if (i < 2 * ts) {
                        ly = TH + 1;
                        lx = i - ts;
                    } else {
                        const int k = i - 2 * ts;
                        ly = 1 + (k >> 1);
                        lx = (k & 1) ? TW + 1 : 0;
                    }
                    tile[ly * ts + lx] =
                        gids[wrapc(y0 + ly - 1, Ly) * Lx + wrapc(x0 + lx - 1, Lx)];
                }
            }
            for (int i = tid; i < ncell; i += nthr) lsa[i] = pa.s_rd[i] + pa.d_rd[i] - A[i];
            // side work of pass P for this tile's cells
            {
                const size_t n = (size_t)a.total_cells;
                int32_t* s_wr = a.sbuf + (size_t)((P + 1u) & 1u) * n + R.cell_off;
                int32_t* d_clr = a.dbuf + (size_t)((P + 1u) % 3u) * n + R.cell_off;
                for (int i = c0 + tid; i < c1; i += nthr) {
                    s_wr[i] = pa.s_rd[i] + pa.d_rd[i];
                    d_clr[i] = 0;
                }
            }
            __syncthreads();
            // the colour's quads of the tile: four consecutive same-colour
            // sites of a row share Philox block k >> 2 (global counters)
            const int cy = c >> 1, cx = c & 1;
            for (int it = tid; it < nq; it += nthr) {
                const int rr = it / (TW >> 3), qi = it - rr * (TW >> 3);
                const int gy = y0 + 2 * rr + cy;
                const int gx0 = x0 + 8 * qi;
                const uint32_t kq = (uint32_t)((gy >> 1) * Q + (gx0 >> 3));
                uint32_t w[4];
                philox4x32_10(kq, p, R.rid, kTagMain, a.key0, a.key1, w);
                const int ly = gy - y0 + 1;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int lx = gx0 - x0 + 2 * u + cx + 1;
                    const int32_t* ru = tile + (ly - 1) * ts;
                    const int32_t* ry = tile + ly * ts;
                    const int32_t* rd = tile + (ly + 1) * ts;
                    const int nb[8] = {ru[lx - 1], ru[lx], ru[lx + 1], ry[lx - 1], ry[lx + 1],
                                       rd[lx - 1], rd[lx], rd[lx + 1]};
                    const int s = ry[lx];
                    const int tg = cpm_decide(a, R, nb, s, w[u], 4u * kq + (uint32_t)u, p, qthr,
                                              lsa, lty, ljs);
                    if (tg >= 0) {
                        tile[ly * ts + lx] = tg;
                        atomicAdd(&pa.d_wr[tg], 1);
                        atomicAdd(&pa.d_wr[s], -1);
                    }
                }
            }
            __syncthreads();
            // the tile's border cells for the neighbouring tiles
            for (int i = tid; i < 2 * TW + 2 * (TH - 2); i += nthr) {
                int ly, lx;
                if (i < TW) {
                    ly = 1;
                    lx = 1 + i;
                } else if (i < 2 * TW) {
                    ly = TH;
                    lx = 1 + i - TW;
                } else {
                    const int k = i - 2 * TW;
                    ly = 2 + (k >> 1);
                    lx = (k & 1) ? TW : 1;
                }
                gids[(y0 + ly - 1) * Lx + x0 + lx - 1] = tile[ly * ts + lx];
            }
            cpm_wait_stores();
            __syncthreads();
            if (tid == 0)
                go = cpm_tile_barrier(bar + r, (uint32_t)n_tiles * (j + 1u), abort_flag);
            __syncthreads();
            if (!go) return;  // uniform: the whole workgroup leaves
        }
    }
    // the tile's interior (its border is already in place)
    for (int i = tid; i < TH * TW; i += nthr) {
        const int ly = 1 + i / TW, lx = 1 + i % TW;
        gids[(y0 + ly - 1) * Lx + x0 + lx - 1] = tile[ly * ts + lx];
    }
}

size_t cpm_tiled_lds_bytes(int tab_lds_bytes, int cell_cap, int TH, int TW) {
    return (size_t)tab_lds_bytes + (size_t)4 * cell_cap + (size_t)((cell_cap + 15) & ~15) +
           (size_t)4 * (TH + 2) * (TW + 2);
}

hipError_t cpm_tiled_occupancy(int tab_lds_bytes, int cell_cap, int TH, int TW, int* per_cu) {
    const size_t lds = cpm_tiled_lds_bytes(tab_lds_bytes, cell_cap, TH, TW);
    hipError_t e = hipFuncSetAttribute((const void*)k_cpm_tiled,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, (const void*)k_cpm_tiled, 256, lds);
}

hipError_t launch_cpm_tiled(const CpmArgs& a, int n_steps, int TH, int TW, int tab_lds_bytes,
                            int cell_cap, int n_blocks, uint32_t* bar, uint32_t* abort_flag,
                            hipStream_t s) {
    const size_t lds = cpm_tiled_lds_bytes(tab_lds_bytes, cell_cap, TH, TW);
    hipLaunchKernelGGL(k_cpm_tiled, dim3(n_blocks), dim3(256), lds, s, a, n_steps, TH, TW,
                       tab_lds_bytes, cell_cap, bar, abort_flag);
    return hipGetLastError();
}

namespace {
// Deciding lanes: one per Philox block of a pass, whole waves; as many drawing
// lanes beside them up to 512.
int cpm_resident_lanes(int range, int max_sites) {
    const int blk = (max_sites / (range == 2 ? 9 : 4) + 3) / 4;
    return blk >= 1024 ? 1024 : (blk + 63) & ~63;
}
}  // namespace

size_t cpm_resident_lds_bytes(int range, int tab_lds_bytes, int cell_cap, int max_sites,
                              int max_padded) {
    const int lanes = cpm_resident_lanes(range, max_sites);
    return (size_t)tab_lds_bytes + (size_t)20 * cell_cap +
           (size_t)(lanes <= 512 ? 16 + 48 : 16) * lanes + (size_t)4 * max_padded;
}

hipError_t launch_cpm_resident(const CpmArgs& a, bool rows, int n_steps, int sw0, int re,
                               int tab_lds_bytes, int cell_cap, int max_sites, int max_padded,
                               hipStream_t s) {
    const size_t lds =
        cpm_resident_lds_bytes(a.range, tab_lds_bytes, cell_cap, max_sites, max_padded);
    const int lanes = cpm_resident_lanes(a.range, max_sites);
    const bool gen = lanes <= 512;
    const void* fn =
        a.range == 2 ? (gen ? (const void*)k_cpm_resident<2, true, false>
                            : (const void*)k_cpm_resident<2, false, false>)
        : rows       ? (gen ? (const void*)k_cpm_resident<1, true, true>
                            : (const void*)k_cpm_resident<1, false, true>)
                     : (gen ? (const void*)k_cpm_resident<1, true, false>
                            : (const void*)k_cpm_resident<1, false, false>);
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    int queue_words = 4 * lanes;
    CpmArgs b = a;
    void* args[] = {&b, &n_steps, &sw0, &re, &tab_lds_bytes, &cell_cap, &queue_words};
    return hipLaunchKernel(fn, dim3(a.R), dim3(gen ? 2 * lanes : lanes), args, lds, s);
}

__global__ void k_cpm_copy(const int32_t* src, int32_t* dst, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        dst[i] = src[i];
}

__device__ __forceinline__ uint64_t first_pass(const CpmArgs& a, int sweep_off) {
    return (uint64_t)(a.range == 2 ? 9 : 4) * (*a.t_base + (uint64_t)sweep_off);
}

__global__ void k_cpm_pass_init(CpmArgs a, int sweep_off) {
    const uint64_t P = first_pass(a, sweep_off);
    const size_t n = (size_t)a.total_cells;
    int32_t* s_wr = a.sbuf + (size_t)(P & 1u) * n;
    int32_t* d0 = a.dbuf + (size_t)((P + 2u) % 3u) * n;
    int32_t* d1 = a.dbuf + (size_t)(P % 3u) * n;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        s_wr[i] = a.area[i];
        d0[i] = 0;
        d1[i] = 0;
    }
}

__global__ void k_cpm_pass_final(CpmArgs a, int sweep_off) {
    const uint64_t P = first_pass(a, sweep_off);
    const size_t n = (size_t)a.total_cells;
    const int32_t* s_rd = a.sbuf + (size_t)(P & 1u) * n;
    const int32_t* d_rd = a.dbuf + (size_t)((P + 2u) % 3u) * n;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        a.area[i] = s_rd[i] + d_rd[i];
}

// Areas from the lattice (after set_state), added into area, which the caller
// cleared: per tile in LDS (cell_cap entries), the medium by wave ballots, then
// one atomic per cell of the tile.  cell_cap = 0 (more cells than LDS holds):
// one atomic per site.  (8 x 512^2, 1000 cells: one atomic per site 1890 us,
// almost all on the medium's word; now 14.)
__global__ void k_cpm_area_count(CpmArgs a, int cell_cap) {
    extern __shared__ int32_t lcnt[];
    const TileDev T = a.tiles[blockIdx.x];
    const RepDev R = a.reps[T.rep];
    const int32_t* ids = a.lat + R.lat_off;
    int32_t* area = a.area + R.cell_off;
    const int n = T.rows * R.Lx;
    const size_t base = (size_t)T.y0 * R.Lx;
    if (cell_cap == 0) {
        for (int i = threadIdx.x; i < n; i += blockDim.x) atomicAdd(&area[ids[base + i]], 1);
        return;
    }
    for (int i = threadIdx.x; i <= R.q; i += blockDim.x) lcnt[i] = 0;
    __syncthreads();
    int medium = 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const int id = ids[base + i];
        if (id == 0)
            ++medium;
        else
            atomicAdd(&lcnt[id], 1);
    }
    medium = __ockl_wfred_add_i32(medium);
    if ((threadIdx.x & 63) == 0 && medium != 0) atomicAdd(&lcnt[0], medium);
    __syncthreads();
    for (int i = threadIdx.x; i <= R.q; i += blockDim.x)
        if (lcnt[i] != 0) atomicAdd(&area[i], lcnt[i]);
}

// Statistics: boundary bonds by type pair (von Neumann, right and down) and
// the adhesion energy over Moore pairs counted once (right, down,
// down-right, down-left), in fixed point; the area term is added by
// k_cpm_area_energy.  stats row: [10 pair counts, H lo, H hi, ...].
__global__ void __launch_bounds__(256) k_cpm_stats(CpmArgs a, int rec_row) {
    __shared__ int32_t ljs[kMaxCpmTypes * kMaxCpmTypes];
    __shared__ int lpair[10];
    __shared__ unsigned long long lH;
    const TileDev T = a.tiles[blockIdx.x];
    const RepDev R = a.reps[T.rep];
    const int nt = R.n_types;
    for (int i = threadIdx.x; i < nt * nt; i += blockDim.x) ljs[i] = a.js[R.js_off + i];
    if (threadIdx.x < 10) lpair[threadIdx.x] = 0;
    if (threadIdx.x == 0) lH = 0ull;
    __syncthreads();
    const int Lx = R.Lx, Ly = R.Ly;
    const int32_t* ids = a.lat + R.lat_off;
    const int8_t* ty = a.ctype + R.cell_off;
    long long H = 0;
    const int n = T.rows * Lx;
    for (int it = threadIdx.x; it < n; it += blockDim.x) {
        const int y = T.y0 + it / Lx, x = it % Lx;
        const int yp = wrapc(y + 1, Ly), xp = wrapc(x + 1, Lx), xm = wrapc(x - 1, Lx);
        const int s = ids[(size_t)y * Lx + x];
        const int ts = ty[s];
        const int r = ids[(size_t)y * Lx + xp], d = ids[(size_t)yp * Lx + x];
        const int dr = ids[(size_t)yp * Lx + xp], dl = ids[(size_t)yp * Lx + xm];
        if (r != s) {
            int p0 = ts, p1 = ty[r];
            if (p0 > p1) { const int tmp = p0; p0 = p1; p1 = tmp; }
            atomicAdd(&lpair[p0 * nt - p0 * (p0 - 1) / 2 + (p1 - p0)], 1);
            H += ljs[ts * nt + ty[r]];
        }
        if (d != s) {
            int p0 = ts, p1 = ty[d];
            if (p0 > p1) { const int tmp = p0; p0 = p1; p1 = tmp; }
            atomicAdd(&lpair[p0 * nt - p0 * (p0 - 1) / 2 + (p1 - p0)], 1);
            H += ljs[ts * nt + ty[d]];
        }
        if (dr != s) H += ljs[ts * nt + ty[dr]];
        if (dl != s) H += ljs[ts * nt + ty[dl]];
        if (a.range == 2) {
            // the second shell's forward half: (0,2), (1,+-2), (2,-2..2)
            const int x2 = wrapc(x + 2, Lx), xm2 = wrapc(x - 2, Lx), y2 = wrapc(y + 2, Ly);
            const int o[8] = {ids[(size_t)y * Lx + x2],   ids[(size_t)yp * Lx + xm2],
                              ids[(size_t)yp * Lx + x2],  ids[(size_t)y2 * Lx + xm2],
                              ids[(size_t)y2 * Lx + xm],  ids[(size_t)y2 * Lx + x],
                              ids[(size_t)y2 * Lx + xp],  ids[(size_t)y2 * Lx + x2]};
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (o[j] != s) H += ljs[ts * nt + ty[o[j]]];
        }
    }
    atomicAdd(&lH, (unsigned long long)H);
    __syncthreads();
    int32_t* row = a.stats + ((size_t)rec_row * a.R + T.rep) * a.width;
    if (threadIdx.x < 10 && lpair[threadIdx.x]) atomicAdd(&row[threadIdx.x], lpair[threadIdx.x]);
    if (threadIdx.x == 0) atomicAdd(reinterpret_cast<unsigned long long*>(row + 10), lH);
}

// lambda S sum over cells (not the medium) of (a - A)^2, one block per replica.
__global__ void k_cpm_area_energy(CpmArgs a, int rec_row) {
    __shared__ unsigned long long lH;
    const int r = blockIdx.x;
    const RepDev R = a.reps[r];
    if (threadIdx.x == 0) lH = 0ull;
    __syncthreads();
    const int32_t* area = a.area + R.cell_off;
    const int32_t* A = a.target + R.cell_off;
    long long H = 0;
    for (int i = 1 + threadIdx.x; i <= R.q; i += blockDim.x) {
        const long long d = (long long)area[i] - (long long)A[i];
        H += R.LS * d * d;
    }
    atomicAdd(&lH, (unsigned long long)H);
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t* row = a.stats + ((size_t)rec_row * a.R + r) * a.width;
        atomicAdd(reinterpret_cast<unsigned long long*>(row + 10), lH);
    }
}

hipError_t launch_cpm_pass(const CpmArgs& a, int n_tiles, int c, int sweep_off, int threads,
                           size_t lds_tab_bytes, hipStream_t s) {
    hipLaunchKernelGGL(k_cpm_pass, dim3(n_tiles), dim3(threads), lds_tab_bytes, s, a, c,
                       sweep_off);
    return hipGetLastError();
}

hipError_t launch_cpm_pass5(const CpmArgs& a, int n_tiles, int c, int sweep_off, int threads,
                            size_t lds_tab_bytes, hipStream_t s) {
    hipLaunchKernelGGL(k_cpm_pass5, dim3(n_tiles), dim3(threads), lds_tab_bytes, s, a, c,
                       sweep_off);
    return hipGetLastError();
}

size_t cpm_quad_lds_bytes(int tab_lds_bytes, int cell_cap) {
    return (size_t)tab_lds_bytes + (size_t)cell_cap * 9;
}

hipError_t launch_cpm_pass_quad(const CpmArgs& a, int n_tiles, int c, int sweep_off,
                                int threads, int tab_lds_bytes, int cell_cap, hipStream_t s) {
    const size_t lds = cpm_quad_lds_bytes(tab_lds_bytes, cell_cap);
    if (threads > 256)
        hipLaunchKernelGGL(k_cpm_pass_site, dim3(n_tiles), dim3(threads), lds, s, a, c, sweep_off,
                           tab_lds_bytes, cell_cap);
    else
        hipLaunchKernelGGL(k_cpm_pass_quad, dim3(n_tiles), dim3(threads), lds, s, a, c, sweep_off,
                           tab_lds_bytes, cell_cap);
    return hipGetLastError();
}

hipError_t cpm_reserve_lds(size_t lds_bytes) {
    hipError_t e = hipFuncSetAttribute((const void*)k_cpm_pass_quad,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)k_cpm_pass_site,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    return e;
}

hipError_t launch_cpm_snapshot(const CpmArgs& a, int total_cells, hipStream_t s) {
    int blocks = (total_cells + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(k_cpm_copy, dim3(blocks), dim3(256), 0, s, a.area, a.snap, total_cells);
    return hipGetLastError();
}

hipError_t launch_cpm_pass_init(const CpmArgs& a, int sweep_off, hipStream_t s) {
    int blocks = (a.total_cells + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(k_cpm_pass_init, dim3(blocks), dim3(256), 0, s, a, sweep_off);
    return hipGetLastError();
}

hipError_t launch_cpm_pass_final(const CpmArgs& a, int sweep_off, hipStream_t s) {
    int blocks = (a.total_cells + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(k_cpm_pass_final, dim3(blocks), dim3(256), 0, s, a, sweep_off);
    return hipGetLastError();
}

hipError_t launch_cpm_area_recount(const CpmArgs& a, int n_tiles, int total_cells, int cell_cap,
                                   hipStream_t s) {
    hipError_t e = launch_fill_i32(a.area, (size_t)total_cells, 0, s);
    if (e != hipSuccess) return e;
    const int cap = cell_cap <= 16384 ? cell_cap : 0;
    hipLaunchKernelGGL(k_cpm_area_count, dim3(n_tiles), dim3(256), (size_t)4 * cap, s, a, cap);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_cpm_snapshot(a, total_cells, s);
}

hipError_t launch_cpm_stats(const CpmArgs& a, int n_tiles, int rec_row, hipStream_t s) {
    hipLaunchKernelGGL(k_cpm_stats, dim3(n_tiles), dim3(256), 0, s, a, rec_row);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_cpm_area_energy, dim3(a.R), dim3(256), 0, s, a, rec_row);
    return hipGetLastError();
}

}  // namespace spinmc
