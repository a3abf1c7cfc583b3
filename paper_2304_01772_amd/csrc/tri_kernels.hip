// Triangular-lattice Ising (the triangular kernels of the Methods): the
// checkerboard Metropolis chain of Algorithm 1 on the six-neighbour lattice.
//
// Sites sit on an Ly x Lx lattice of int8 spins; the neighbours of (y, x)
// are (y, x+-1), (y+-1, x), (y-1, x+1) and (y+1, x-1) (periodic), one
// coupling J for every bond, H = -J sum s s' - h sum s.  Three colours
// c = (x + 2y) mod 3 -- no bond joins two sites of one colour when Lx and Ly
// are multiples of 3 -- make a sweep of three passes p = 3t + c.  The sites
// of colour c in row y are x = 3i + (c + y) mod 3; on the device each colour
// has a plane of Ly rows of Lx/3 bytes, site (y, x) at byte (y, x / 3) of
// plane (x + 2y) mod 3, so that byte k of plane c is the site with
// within-colour index k = y Lx/3 + i.  It selects word k & 3 of Philox4x32-10
// block (k >> 2, p, rid, 0), used whole as W; the flip is accepted iff
// W < T[7 [s > 0] + (S6 + 6) / 2] with the FP64 host thresholds
// T = ceil(2^32 exp(-beta 2 s (J S6 + h))) (2^32 when that change is <= 0).
// A lane takes the four sites of one Philox block.
#include "tri_internal.hpp"

namespace spinmc {

namespace {
constexpr uint32_t kTriTagMain = 0u, kTriTagInit = 2u;

__device__ __forceinline__ int wrapt(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// Byte of site (y, x) of a triangular lattice in its colour planes.
__device__ __forceinline__ size_t tri_byte(int y, int x, int Lx, int Ly) {
    const size_t W3 = (size_t)(Lx / 3);
    return (size_t)((x + 2 * y) % 3) * Ly * W3 + (size_t)y * W3 + (size_t)(x / 3);
}

// Chain / square / cubic lattices sit in two colour planes on the device:
// site (z, y, x) of row z Ly + y is byte (row, x >> 1) of plane
// (x + y + z) & 1, each plane Ly Lz rows of W = Lx / 2 bytes.  The byte's
// offset in its plane is the site's within-colour index k = (row Lx + x) >> 1.
__device__ __forceinline__ size_t hc_byte(int z, int y, int x, int Lx, int Ly, int Lz) {
    const size_t W = (size_t)(Lx >> 1);
    return (size_t)((x + y + z) & 1) * Ly * Lz * W + ((size_t)z * Ly + y) * W + (x >> 1);
}
}  // namespace

// Initial spins from the init stream of the Ising model: site n = y Lx + x
// takes word n & 3 of block (n >> 2, 0, rid, 2); +1 iff it is < 2^31.
__global__ void __launch_bounds__(256) k_tri_init(TriArgs a) {
    const RepDev D = a.reps[blockIdx.y];
    const int n = D.Lx * D.Ly * (D.model == kModelIsingHC ? D.q : 1);
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (4 * b >= n) return;
    uint32_t w[4];
    philox4x32_10((uint32_t)b, 0u, D.rid, kTriTagInit, a.key0, a.key1, w);
    int8_t* lat = a.lat + D.lat_off;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int i = 4 * b + u;
        if (i >= n) break;
        const int8_t v = w[u] < 0x80000000u ? (int8_t)1 : (int8_t)-1;
        if (D.model == kModelIsingHC) {
            const int row = i / D.Lx, x = i - row * D.Lx, z = row / D.Ly;
            lat[hc_byte(z, row - z * D.Ly, x, D.Lx, D.Ly, D.q)] = v;
        } else {
            const int y = i / D.Lx;
            lat[tri_byte(y, i - y * D.Lx, D.Lx, D.Ly)] = v;
        }
    }
}

// Span form of a pass (four sites of one Philox block per lane, byte
// arithmetic in 32-bit words).  A spin byte is 0x01 (+1) or 0xFF (-1), so
// v & 0x02020202 flags the -1 bytes of a word as 2 per byte.  Sums of such
// flags stay below 16 per byte (at most six neighbours), so whole words add
// without carries between bytes: one add chain gives 2n, n the number of -1
// neighbours, at every byte position of a span.  The threshold class
// 7 [s > 0] + (S + 6) / 2 (S the neighbour sum over the k neighbours present,
// S = k - 2n) is then keyed by j = n + 8 [s < 0], read from a 16-entry table.
namespace {
constexpr uint32_t kNegFlag = 0x02020202u;

__device__ __forceinline__ uint32_t abyte(uint32_t hi, uint32_t lo, uint32_t sel) {
    return __builtin_amdgcn_alignbyte(hi, lo, sel);  // ({hi, lo} >> 8 sel)[31:0]
}

// entry j = n + 8 neg of the keyed table from the 14 classes, k neighbours
__device__ __forceinline__ uint64_t keyed_threshold(const uint64_t* tab, int j, int k) {
    const int n = j & 7, neg = j >> 3;
    return n > k ? 0ull : tab[7 * (1 - neg) + (k + 6) / 2 - n];
}

// Chain / square / cubic on the colour planes: S the four own bytes (plane
// bytes j0 .. j0 + 3 of a row, own sites x = 2 j + par), N the added -1 flags
// of the vertical partners (the other plane's rows y +- 1 and z +- 1, same
// bytes), M the other plane's word of the same row and hf the -1 flag of its
// halo byte (j0 - 1 for par = 0, j0 + 4 for par = 1): the horizontal partners
// of own byte j are the other plane's bytes j - 1 + par and j + par.
__device__ __forceinline__ uint32_t hc_word(uint32_t S, uint32_t N, uint32_t M, uint32_t hf,
                                            uint32_t par, const uint32_t (&w)[4],
                                            const uint64_t* lt) {
    const uint32_t mf = M & kNegFlag;
    const uint32_t H = mf + (par ? abyte(hf, mf, 1) : abyte(mf, hf << 24, 3));
    const uint32_t K = (N + H) | ((S & kNegFlag) << 3);  // 2n + 16 [s < 0] per byte
    uint32_t F = 0u;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        F |= (uint64_t)w[u] < lt[(K >> (8 * u + 1)) & 15u] ? 0xFEu << (8 * u) : 0u;
    return S ^ F;  // a flip negates the byte: s -> -s is s ^ 0xFE for s = +-1
}

// b / d for 0 <= b < 2^22, d >= 1: the FP32 estimate b (1/d) is within one
// of the quotient there (relative error below 2^-22), one correction each way
__device__ __forceinline__ int qdiv(int b, int d, bool small) {
    if (!small) return b / d;
    int q = (int)((float)b * __builtin_amdgcn_rcpf((float)d));
    const int rem = b - (int)__umul24((uint32_t)q, (uint32_t)d);
    q += rem >= d ? 1 : 0;
    q -= rem < 0 ? 1 : 0;
    return q;
}

// Workgroup w of a 1-D grid of n runs on XCD w mod 8 (round-robin
// dispatch); the logical index (w mod 8) n/8 + w/8 keeps consecutive logical
// workgroups -- neighbouring spans of one replica -- on one XCD and its L2.
__device__ __forceinline__ int xcd_logical(int w, int n) {
    return (n & 7) ? w : (w & 7) * (n >> 3) + (w >> 3);
}

__device__ __forceinline__ uint32_t ld32(const int8_t* p) { return *reinterpret_cast<const uint32_t*>(p); }
__device__ __forceinline__ uint2 ld64(const int8_t* p) { return *reinterpret_cast<const uint2*>(p); }
__device__ __forceinline__ uint32_t negflag(const int8_t* p) { return (uint32_t)(uint8_t)*p & 2u; }
}  // namespace

// Lattices of any width, site by site on the colour planes.  A lane takes the four
// sites of a Philox block, which may run on into the next rows: one division finds
// the first, the others follow by steps, and all of the block's bytes are loaded
// before any is decided.  Bound by its byte loads (28 a block in three dimensions)
// and their addresses; with one division a site and each site's loads behind the
// store before it, 4 triangular lattices of 195^2 took 13.1 us a sweep, 8 x 375^2
// 14.9, now 11.2 and 12.5; a recorded sweep 26 us more, now 6.
namespace {
template <int MODEL>
struct PlaneSite {
    int W, Ly, Lz, nk;
    int row, j, y, z;  // the site is byte j of row z Ly + y of its plane

    __device__ __forceinline__ PlaneSite(const RepDev& D, int k) {
        constexpr bool TRI = MODEL == kModelIsingTri;
        W = TRI ? D.Lx / 3 : D.Lx >> 1;
        Ly = D.Ly;
        Lz = TRI ? 1 : D.q;
        nk = W * Ly * Lz;
        const bool small = nk < 1 << 22;
        row = qdiv(k, W, small);
        j = k - row * W;
        z = Lz > 1 ? qdiv(row, Ly, small) : 0;
        y = row - z * Ly;
    }
    __device__ __forceinline__ void step() {  // to the next site, staying on the last
        const bool last = row * W + j + 1 >= nk;
        const bool nr = j + 1 == W && !last, ns = nr && y + 1 == Ly;
        j = nr ? 0 : (last ? j : j + 1);
        row += nr ? 1 : 0;
        y = ns ? 0 : (nr ? y + 1 : y);
        z += ns ? 1 : 0;
    }
    // x of the site is (2 or 3) j + phase
    __device__ __forceinline__ int phase(int c) const {
        return MODEL == kModelIsingTri ? (c + y) % 3 : (c + y + z) & 1;
    }
    // places in the partners' planes of x + 1 and x - 1 in this row, and the steps to
    // the rows around it
    __device__ __forceinline__ int right(int ph) const {
        return row * W + (ph != (MODEL == kModelIsingTri ? 2 : 1) ? j : (j + 1 == W ? 0 : j + 1));
    }
    __device__ __forceinline__ int left(int ph) const {
        return row * W + (ph != 0 ? j : (j == 0 ? W - 1 : j - 1));
    }
    __device__ __forceinline__ int up() const { return y == 0 ? (Ly - 1) * W : -W; }
    __device__ __forceinline__ int down() const { return y + 1 == Ly ? (1 - Ly) * W : W; }
    __device__ __forceinline__ int zup() const { return (z == 0 ? Lz - 1 : -1) * Ly * W; }
    __device__ __forceinline__ int zdown() const { return (z + 1 == Lz ? 1 - Lz : 1) * Ly * W; }
};
}  // namespace

template <int MODEL>
__global__ void __launch_bounds__(256) k_plane_pass_any(TriArgs a, int c, int sweep_off) {
    __shared__ uint64_t lt[kTriClasses];
    constexpr bool TRI = MODEL == kModelIsingTri;
    const int r = blockIdx.y;
    if (threadIdx.x < kTriClasses) lt[threadIdx.x] = a.tab[(size_t)r * kTriClasses + threadIdx.x];
    __syncthreads();
    const RepDev D = a.reps[r];
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    const int nk = (TRI ? D.Lx / 3 : D.Lx >> 1) * D.Ly * (TRI ? 1 : D.q);
    if (4 * b >= nk) return;
    PlaneSite<MODEL> q(D, 4 * b);
    int8_t* own = a.lat + D.lat_off + (size_t)c * nk;
    // the planes of the next colour and of the one before (one plane with two colours)
    const int8_t* nx = a.lat + D.lat_off + (size_t)(TRI ? (c + 1) % 3 : 1 - c) * nk;
    const int8_t* pv = a.lat + D.lat_off + (size_t)(TRI ? (c + 2) % 3 : 1 - c) * nk;
    int s[4], S[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int ph = q.phase(c), o = q.row * q.W + q.j, R = q.right(ph), L = q.left(ph);
        s[u] = own[o];
        S[u] = nx[R] + pv[L];
        if (TRI)
            S[u] += nx[o + q.up()] + pv[o + q.down()] + pv[R + q.up()] + nx[L + q.down()];
        else {
            if (q.Ly > 1) S[u] += nx[o + q.up()] + nx[o + q.down()];
            if (q.Lz > 1) S[u] += nx[o + q.zup()] + nx[o + q.zdown()];
        }
        q.step();
    }
    const uint64_t t = *a.t_base + (uint64_t)sweep_off;
    uint32_t w[4];
    philox4x32_10((uint32_t)b, (uint32_t)((TRI ? 3 : 2) * t + (uint64_t)c), D.rid, kTriTagMain, a.key0,
                  a.key1, w);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int idx = 7 * (s[u] > 0) + (S[u] + 6) / 2;
        if (4 * b + u < nk && (uint64_t)w[u] < lt[idx]) own[4 * b + u] = (int8_t)(-s[u]);
    }
}

// A workgroup's sums of v into row, one atomic a statistic (an atomic a wave of 62
// workgroups of 256 lanes took 25 us, all on one cache line).
__device__ __forceinline__ void add_sums(int (&v)[4], int32_t* row) {
    __shared__ int sum[4];
    if (threadIdx.x < 4) sum[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        for (int o = 32; o > 0; o >>= 1) v[k] += __shfl_xor(v[k], o);
        if ((threadIdx.x & 63) == 0) atomicAdd(&sum[k], v[k]);
    }
    __syncthreads();
    if (threadIdx.x < 4) atomicAdd(&row[threadIdx.x], sum[threadIdx.x]);
}

// [M, B1, B2, B3] of any width (integers, so the order does not matter).
template <int MODEL>
__global__ void __launch_bounds__(256) k_plane_stats_any(TriArgs a, int rec_row) {
    constexpr bool TRI = MODEL == kModelIsingTri;
    constexpr int ncol = TRI ? 3 : 2;
    const int r = blockIdx.y;
    const RepDev D = a.reps[r];
    const int8_t* lat = a.lat + D.lat_off;
    const int nk = (TRI ? D.Lx / 3 : D.Lx >> 1) * D.Ly * (TRI ? 1 : D.q), nb = (nk + 3) >> 2;
    int v[4] = {0, 0, 0, 0};
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < ncol * nb; i += gridDim.x * blockDim.x) {
        const int c = (i >= nb ? 1 : 0) + (TRI && i >= 2 * nb ? 1 : 0), b = i - c * nb;
        const int8_t* own = lat + (size_t)c * nk;
        const int8_t* nx = lat + (size_t)(TRI ? (c + 1) % 3 : 1 - c) * nk;
        const int8_t* pv = lat + (size_t)(TRI ? (c + 2) % 3 : 1 - c) * nk;
        PlaneSite<MODEL> q(D, 4 * b);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int ph = q.phase(c), o = q.row * q.W + q.j;
            const int s = 4 * b + u < nk ? own[o] : 0;
            v[0] += s;
            v[1] += s * nx[q.right(ph)];
            if (TRI) {
                v[2] += s * pv[o + q.down()];
                v[3] += s * nx[q.left(ph) + q.down()];
            } else {
                if (q.Ly > 1) v[2] += s * nx[o + q.down()];
                if (q.Lz > 1) v[3] += s * nx[o + q.zdown()];
            }
            q.step();
        }
    }
    add_sums(v, &a.stats[((size_t)rec_row * a.R + r) * a.width]);
}

// Lx a multiple of 12: the four sites of a Philox block are four consecutive
// bytes i0 .. i0 + 3 of row y of plane c (planes of W3 = Lx / 3 bytes per
// row).  With r = (c + y) mod 3 the six neighbours of own byte i are, in
// plane c + 1: row y at i + [r = 2] (x + 1), row y - 1 at i (y - 1, x) and
// row y + 1 at i - [r = 0] (y + 1, x - 1); in plane c + 2: row y at
// i - [r = 0] (x - 1), row y + 1 at i (y + 1, x) and row y - 1 at
// i + [r = 2] (y - 1, x + 1) -- six dwords, two of them with a halo byte
// on the side of the shift.  Only the own dword is stored.  A lane takes NB
// Philox blocks, 256 apart (a wave's loads of one block index stay
// contiguous), their loads all in flight together: NB = 2 for large passes
// (see launch_tri_pass), 1 otherwise.  The grid is 1-D: gx workgroups per
// replica, replica-major in logical order.
template <int NB>
__global__ void __launch_bounds__(256) k_tri_pass4(TriArgs a, int c, int sweep_off, int gx) {
    __shared__ uint64_t lt[16];
    const int wl = xcd_logical((int)blockIdx.x, (int)gridDim.x);
    const int r = wl / gx, wx = wl - r * gx;
    const RepDev D = a.reps[r];
    const int Lx = D.Lx, Ly = D.Ly, W3 = Lx / 3, qpr = W3 >> 2, nb = Ly * qpr;
    const int bt = NB * wx * 256 + (int)threadIdx.x;  // block k: bt + 256 k
    if (NB * wx * 256 >= nb) return;  // whole workgroup past the end
    const bool small = nb < (1 << 22);
    // 32-bit offsets from the replica's base (a lattice below 2^31 bytes)
    const uint32_t psz = (uint32_t)Ly * (uint32_t)W3;  // bytes per plane
    const int cp = c == 2 ? 0 : c + 1, cm = c == 0 ? 2 : c - 1;
    int8_t* own = a.lat + D.lat_off + (uint32_t)c * psz;
    const int8_t* pp = a.lat + D.lat_off + (uint32_t)cp * psz;
    const int8_t* pm = a.lat + D.lat_off + (uint32_t)cm * psz;
    // blocks past the end compute the last block and store nothing (every
    // lane reaches the barrier)
    uint32_t S[NB], N[NB], off[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const int b = bt + 256 * k < nb ? bt + 256 * k : nb - 1;
        const int y = qdiv(b, qpr, small);
        const int i0 = 4 * (b - (int)__umul24((uint32_t)y, (uint32_t)qpr));
        const int yu = y == 0 ? Ly - 1 : y - 1, yd = y + 1 == Ly ? 0 : y + 1;
        const uint32_t o = __umul24((uint32_t)y, (uint32_t)W3);
        const uint32_t ou = __umul24((uint32_t)yu, (uint32_t)W3);
        const uint32_t od = __umul24((uint32_t)yd, (uint32_t)W3);
        const int rr = (c + y) % 3;
        off[k] = o + (uint32_t)i0;
        S[k] = ld32(own + off[k]);
        const uint32_t fa = ld32(pp + off[k]) & kNegFlag;           // (y, x + 1)
        const uint32_t fb = ld32(pp + (ou + i0)) & kNegFlag;        // (y - 1, x)
        const uint32_t fc = ld32(pp + (od + i0)) & kNegFlag;        // (y + 1, x - 1)
        const uint32_t fd = ld32(pm + off[k]) & kNegFlag;           // (y, x - 1)
        const uint32_t fe = ld32(pm + (od + i0)) & kNegFlag;        // (y + 1, x)
        const uint32_t ff = ld32(pm + (ou + i0)) & kNegFlag;        // (y - 1, x + 1)
        // halo bytes: r = 2 shifts (y, x + 1) and (y - 1, x + 1) by one byte
        // up (byte i0 + 4), r = 0 shifts (y + 1, x - 1) and (y, x - 1) down
        // (byte i0 - 1); r = 1 needs neither
        const int ir = i0 + 4 == W3 ? 0 : i0 + 4, il = i0 == 0 ? W3 - 1 : i0 - 1;
        const uint32_t h1 = negflag(rr == 2 ? pp + (o + ir) : pp + (od + il));
        const uint32_t h2 = negflag(rr == 2 ? pm + (ou + ir) : pm + (o + il));
        const uint32_t sa = rr == 2 ? abyte(h1, fa, 1) : fa;
        const uint32_t sf = rr == 2 ? abyte(h2, ff, 1) : ff;
        const uint32_t sc = rr == 0 ? abyte(fc, h1 << 24, 3) : fc;
        const uint32_t sd = rr == 0 ? abyte(fd, h2 << 24, 3) : fd;
        N[k] = sa + fb + sc + sd + fe + sf;  // 2n per byte, n <= 6 -1 neighbours
    }
    const uint64_t t = *a.t_base + (uint64_t)sweep_off;
    const uint32_t p = (uint32_t)(3 * t + (uint64_t)c);
    uint32_t w[NB][4];
#pragma unroll
    for (int k = 0; k < NB; ++k)
        philox4x32_10((uint32_t)(bt + 256 * k), p, D.rid, kTriTagMain, a.key0, a.key1, w[k]);
    // the table after the loads and the random words: its latency overlaps theirs
    if (threadIdx.x < 16)
        lt[threadIdx.x] = keyed_threshold(a.tab + (size_t)r * kTriClasses, threadIdx.x, 6);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const uint32_t K = N[k] | ((S[k] & kNegFlag) << 3);  // 2n + 16 [s < 0] per byte
        uint32_t F = 0u;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            F |= (uint64_t)w[k][u] < lt[(K >> (8 * u + 1)) & 15u] ? 0xFEu << (8 * u) : 0u;
        if (bt + 256 * k < nb) *reinterpret_cast<uint32_t*>(own + off[k]) = S[k] ^ F;
    }
}

// Lx a multiple of 8: the four sites of a Philox block are four consecutive
// bytes j0 .. j0 + 3 of a row of plane c (plane rows of W = Lx / 2 bytes, so
// a row holds W / 4 blocks); the other plane's word of the same row plus one
// halo byte, and its words of rows y +- 1 and z +- 1, come in as dwords, and
// only the own word is stored.  A lane takes NB Philox blocks, 256 apart, as
// k_tri_pass4.
template <int NB>
__global__ void __launch_bounds__(256) k_hc_pass4(TriArgs a, int c, int sweep_off, int gx) {
    __shared__ uint64_t lt[16];
    const int wl = xcd_logical((int)blockIdx.x, (int)gridDim.x);  // see k_tri_pass4
    const int r = wl / gx, wx = wl - r * gx;
    const RepDev D = a.reps[r];
    const int Lx = D.Lx, Ly = D.Ly, Lz = D.q, W = Lx >> 1, qpr = W >> 2;
    const int nb = Ly * Lz * qpr;  // Philox blocks per pass: Lx Ly Lz / 8
    const int bt = NB * wx * 256 + (int)threadIdx.x;  // block k: bt + 256 k
    if (NB * wx * 256 >= nb) return;  // whole workgroup past the end
    const bool small = nb < (1 << 22);
    // 32-bit offsets from the replica's base (a lattice below 2^31 bytes)
    const uint32_t psz = (uint32_t)(Ly * Lz) * (uint32_t)W;  // bytes per plane
    int8_t* own = a.lat + D.lat_off + (c ? psz : 0u);
    const int8_t* oth = a.lat + D.lat_off + (c ? 0u : psz);
    uint32_t S[NB], N[NB], M[NB], hf[NB], off[NB], par[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const int b = bt + 256 * k < nb ? bt + 256 * k : nb - 1;  // see k_tri_pass4
        const int row = qdiv(b, qpr, small);  // z Ly + y
        const int j0 = 4 * (b - (int)__umul24((uint32_t)row, (uint32_t)qpr));
        const int z = qdiv(row, Ly, small), y = row - (int)__umul24((uint32_t)z, (uint32_t)Ly);
        const uint32_t ro = (uint32_t)row * (uint32_t)W;
        off[k] = ro + (uint32_t)j0;
        par[k] = (uint32_t)((c + y + z) & 1);
        S[k] = ld32(own + off[k]);
        M[k] = ld32(oth + off[k]);
        const int hb = par[k] ? (j0 + 4 == W ? 0 : j0 + 4) : (j0 == 0 ? W - 1 : j0 - 1);
        hf[k] = negflag(oth + (ro + (uint32_t)hb));
        N[k] = 0u;
        if (Ly > 1) {
            const uint32_t zr = (uint32_t)(z * Ly);
            N[k] += (ld32(oth + ((zr + wrapt(y - 1, Ly)) * (uint32_t)W + j0)) & kNegFlag) +
                    (ld32(oth + ((zr + wrapt(y + 1, Ly)) * (uint32_t)W + j0)) & kNegFlag);
        }
        if (Lz > 1) {
            N[k] += (ld32(oth + ((uint32_t)(wrapt(z - 1, Lz) * Ly + y) * (uint32_t)W + j0)) & kNegFlag) +
                    (ld32(oth + ((uint32_t)(wrapt(z + 1, Lz) * Ly + y) * (uint32_t)W + j0)) & kNegFlag);
        }
    }
    const uint64_t t = *a.t_base + (uint64_t)sweep_off;
    const uint32_t p = (uint32_t)(2 * t + (uint64_t)c);
    uint32_t w[NB][4];
#pragma unroll
    for (int k = 0; k < NB; ++k)
        philox4x32_10((uint32_t)(bt + 256 * k), p, D.rid, kTriTagMain, a.key0, a.key1, w[k]);
    if (threadIdx.x < 16)
        lt[threadIdx.x] = keyed_threshold(a.tab + (size_t)r * kTriClasses, threadIdx.x,
                                          2 + 2 * (Ly > 1) + 2 * (Lz > 1));
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const uint32_t v = hc_word(S[k], N[k], M[k], hf[k], par[k], w[k], lt);
        if (bt + 256 * k < nb) *reinterpret_cast<uint32_t*>(own + off[k]) = v;
    }
}

// (e, |m|, m^2, m) per replica from [M, B1, B2, B3] (either lattice).
__global__ void k_tri_observables(TriArgs a, double* obs) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= a.R) return;
    const RepDev D = a.reps[r];
    const int32_t* s = a.stats + (size_t)r * a.width;
    const double N = (double)D.Lx * (double)D.Ly * (D.model == kModelIsingHC ? (double)D.q : 1.0);
    const double M = s[0];
    const double H = -((double)D.Jx * ((double)s[1] + (double)s[2] + (double)s[3]) +
                       (double)D.h * M);
    double* o = obs + (size_t)r * 4;
    o[0] = H / N;
    o[1] = fabs(M) / N;
    o[2] = (M / N) * (M / N);
    o[3] = M / N;
}

// ------------------------------------------------ LDS-resident colour planes
// All sweeps of a call in one launch, one workgroup per replica, its colour
// planes in LDS in the order they have in global memory and a barrier after
// every colour pass: the same decisions as the streamed passes, without the
// per-pass launches and lattice round trips.  A spin is one byte, 1 for -1
// and 0 for +1, so that sums of neighbour words need no masks.
//
// A lane owns NI items for the whole launch; an item is NB consecutive Philox
// blocks of a plane row, 4 NB bytes at the same place of every plane, read as
// one LDS access.  Their offsets are worked out once per launch (they are the
// same in every pass), which leaves a pass the Philox rounds (57 of about 85
// lane-cycles a block), the neighbour words and one table lookup and compare
// per site.  (In natural order, where a 12- or 8-byte span holds four own
// sites, the same passes took about 45 lane-instructions a site: 1024 x 96^2
// triangular, 200 sweeps with every tenth recorded, 2705 us; 256 x 32^3, 100
// sweeps and one measurement, 1000 us; now 982 and 437.)
//
// NB = 2 for lattices of more than 1024 blocks a plane whose rows hold an even
// number of blocks (half the LDS accesses and offsets per site), else 1; NI = 1 up to 1024 items (any number
// of waves, several workgroups to a CU), else up to 8 / NB.
template <int NB>
struct Words {
    uint32_t v[NB];
};

template <int NB>
__device__ __forceinline__ Words<NB> ldw(const int8_t* p) {
    Words<NB> r;
    if (NB == 2) {
        const uint2 t = *reinterpret_cast<const uint2*>(p);
        r.v[0] = t.x;
        r.v[NB - 1] = t.y;
    } else {
        r.v[0] = *reinterpret_cast<const uint32_t*>(p);
    }
    return r;
}

template <int NB>
__device__ __forceinline__ void stw(int8_t* p, const Words<NB>& w) {
    if (NB == 2)
        *reinterpret_cast<uint2*>(p) = make_uint2(w.v[0], w.v[NB - 1]);
    else
        *reinterpret_cast<uint32_t*>(p) = w.v[0];
}

__device__ __forceinline__ uint32_t lbyte(const int8_t* p) { return (uint32_t)(uint8_t)*p; }

// Bytes moved by one place within a row: up takes byte i + 1 (h, its low
// byte, follows the last word) where sh = 1, and leaves w where sh = 0; down
// takes byte i - 1 (h << 24 precedes the first word) under the selector
// kDown, and leaves w under kKeep.
constexpr uint32_t kDown = 0x06050403u, kKeep = 0x07060504u;

template <int NB>
__device__ __forceinline__ Words<NB> bytes_up(const Words<NB>& w, uint32_t h, uint32_t sh) {
    Words<NB> r;
#pragma unroll
    for (int k = 0; k < NB; ++k) r.v[k] = abyte(k + 1 < NB ? w.v[k + 1] : h, w.v[k], sh);
    return r;
}

template <int NB>
__device__ __forceinline__ Words<NB> bytes_down(const Words<NB>& w, uint32_t h, uint32_t sel) {
    Words<NB> r;
#pragma unroll
    for (int k = 0; k < NB; ++k)
        r.v[k] = __builtin_amdgcn_perm(w.v[k], k > 0 ? w.v[k - 1] : h << 24, sel);
    return r;
}

// An item's place: off the offset of its first byte within a plane, ou / od
// the same bytes of rows y - 1 / y + 1, ozu / ozd of planes z - 1 / z + 1
// (chain / cubic), dl / dr from off to the bytes left and right of it (row
// ends wrap), ph its row's phase (y mod 3, or (y + z) mod 2).
struct PlaneItem {
    uint32_t off, ou, od, ozu, ozd;
    int dl, dr;
    uint32_t ph;
};

// The same in four registers (a plane of an LDS-resident lattice is at most
// 32 KiB, so every offset fits 15 bits): what a lane keeps of each item when
// it owns several.
struct PackedItem {
    uint32_t a, b, c, d;
};

__device__ __forceinline__ PackedItem pack_item(const PlaneItem& t) {
    return PackedItem{t.off | (t.ph << 16), t.ou | (t.od << 16), t.ozu | (t.ozd << 16),
                      ((uint32_t)t.dl & 0xFFFFu) | ((uint32_t)t.dr << 16)};
}

__device__ __forceinline__ PlaneItem unpack_item(PackedItem p) {
    // opaque here, so that the unpacked values of all items are not kept
    // over the whole sweep loop
    asm volatile("" : "+v"(p.a), "+v"(p.b), "+v"(p.c), "+v"(p.d));
    PlaneItem t;
    t.off = p.a & 0xFFFFu;
    t.ph = p.a >> 16;
    t.ou = p.b & 0xFFFFu;
    t.od = p.b >> 16;
    t.ozu = p.c & 0xFFFFu;
    t.ozd = p.c >> 16;
    t.dl = (int)(int16_t)(p.d & 0xFFFFu);
    t.dr = (int)p.d >> 16;
    return t;
}

template <int MODEL, int NB>
__device__ __forceinline__ PlaneItem plane_item(int i, int Lx, int Ly, int Lz) {
    PlaneItem t;
    const int W = MODEL == kModelIsingTri ? Lx / 3 : Lx >> 1, G = W / (4 * NB);
    const int row = i / G, j = 4 * NB * (i - row * G);
    const int z = row / Ly, y = row - z * Ly;
    const int yu = y == 0 ? Ly - 1 : y - 1, yd = y + 1 == Ly ? 0 : y + 1;
    t.off = (uint32_t)(row * W + j);
    t.ou = (uint32_t)((z * Ly + yu) * W + j);
    t.od = (uint32_t)((z * Ly + yd) * W + j);
    t.ozu = (uint32_t)(((z == 0 ? Lz - 1 : z - 1) * Ly + y) * W + j);
    t.ozd = (uint32_t)(((z + 1 == Lz ? 0 : z + 1) * Ly + y) * W + j);
    t.dl = j == 0 ? W - 1 : -1;
    t.dr = j + 4 * NB == W ? -j : 4 * NB;
    t.ph = MODEL == kModelIsingTri ? (uint32_t)(y % 3) : (uint32_t)((y + z) & 1);
    return t;
}

// The six neighbours of the item's colour-c sites (see k_tri_pass4): row
// phase rr = (c + y) mod 3 decides which of the words move by a byte.
template <int NB>
struct TriWords {
    Words<NB> S, sa, fb, sc, sd, fe, sf;
};

template <int NB, bool ALL>
__device__ __forceinline__ TriWords<NB> tri_words(const int8_t* ls, uint32_t psz, int c,
                                                  const PlaneItem& t) {
    const int cp = c == 2 ? 0 : c + 1, cm = c == 0 ? 2 : c - 1;
    const int8_t* own = ls + (uint32_t)c * psz;
    const int8_t* pp = ls + (uint32_t)cp * psz;
    const int8_t* pm = ls + (uint32_t)cm * psz;
    const uint32_t r = t.ph + (uint32_t)c, rr = r >= 3u ? r - 3u : r;
    const bool up = rr == 2u, dn = rr == 0u;
    const uint32_t sh = up ? 1u : 0u, sel = dn ? kDown : kKeep;
    TriWords<NB> w;
    w.S = ldw<NB>(own + t.off);
    const Words<NB> fa = ldw<NB>(pp + t.off), fc = ldw<NB>(pp + t.od);
    w.fe = ldw<NB>(pm + t.od);
    const uint32_t h1 = lbyte(pp + (up ? t.off + (uint32_t)t.dr : t.od + (uint32_t)t.dl));
    w.sa = bytes_up<NB>(fa, h1, sh);
    w.sc = bytes_down<NB>(fc, h1, sel);
    if (ALL) {
        w.fb = ldw<NB>(pp + t.ou);
        const Words<NB> fd = ldw<NB>(pm + t.off), ff = ldw<NB>(pm + t.ou);
        const uint32_t h2 = lbyte(pm + (up ? t.ou + (uint32_t)t.dr : t.off + (uint32_t)t.dl));
        w.sd = bytes_down<NB>(fd, h2, sel);
        w.sf = bytes_up<NB>(ff, h2, sh);
    }
    return w;
}

// The horizontal neighbours of the item's colour-c sites: the other plane's
// own bytes M and those moved towards the side of the row's parity.
template <int NB>
__device__ __forceinline__ void hc_words(const int8_t* oth, int c, const PlaneItem& t,
                                         Words<NB>& M, Words<NB>& H) {
    const bool par = ((t.ph + (uint32_t)c) & 1u) != 0u;
    M = ldw<NB>(oth + t.off);
    const uint32_t h = lbyte(oth + (t.off + (uint32_t)(par ? t.dr : t.dl)));
    // byte i + 1 (par) or i - 1: the neighbouring word on that side, one perm
    const uint32_t sel = par ? 0x00070605u : kDown;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const uint32_t nx = k + 1 < NB ? M.v[k + 1] : h, pv = k > 0 ? M.v[k - 1] : h << 24;
        H.v[k] = __builtin_amdgcn_perm(M.v[k], par ? nx : pv, sel);
    }
}

// Adds to cnt an item's -1 spins and unequal bonds in each direction, from
// bytes whose bits MASK tell the spins apart: triangular from every site's three
// forward bonds, chain / cubic from both ends' directions of the colour-1 sites
// (every bond has one colour-1 end) and the spins of both colours.
template <int MODEL, int NB, uint32_t MASK>
__device__ __forceinline__ void count_item(const int8_t* ls, uint32_t psz, const PlaneItem& q,
                                           int Ly, int Lz, int (&cnt)[4]) {
    if (MODEL == kModelIsingTri) {
        for (int c = 0; c < 3; ++c) {
            const TriWords<NB> w = tri_words<NB, false>(ls, psz, c, q);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const uint32_t s = w.S.v[b];
                cnt[0] += __popc(s & MASK);
                cnt[1] += __popc((s ^ w.sa.v[b]) & MASK);
                cnt[2] += __popc((s ^ w.fe.v[b]) & MASK);
                cnt[3] += __popc((s ^ w.sc.v[b]) & MASK);
            }
        }
    } else {
        Words<NB> M, H;
        hc_words<NB>(ls, 1, q, M, H);
        const Words<NB> S = ldw<NB>(ls + psz + q.off);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            cnt[0] += __popc(S.v[b] & MASK) + __popc(M.v[b] & MASK);
            cnt[1] += __popc((S.v[b] ^ M.v[b]) & MASK) + __popc((S.v[b] ^ H.v[b]) & MASK);
        }
        if (Ly > 1) {
            const Words<NB> u = ldw<NB>(ls + q.ou), d = ldw<NB>(ls + q.od);
#pragma unroll
            for (int b = 0; b < NB; ++b)
                cnt[2] += __popc((S.v[b] ^ u.v[b]) & MASK) + __popc((S.v[b] ^ d.v[b]) & MASK);
        }
        if (Lz > 1) {
            const Words<NB> u = ldw<NB>(ls + q.ozu), d = ldw<NB>(ls + q.ozd);
#pragma unroll
            for (int b = 0; b < NB; ++b)
                cnt[3] += __popc((S.v[b] ^ u.v[b]) & MASK) + __popc((S.v[b] ^ d.v[b]) & MASK);
        }
    }
}

// [M, B1, B2, B3] of lattices in memory, rows of whole Philox blocks (Lx % 12 == 0
// triangular, % 8 == 0 chain / cubic): items of 4 NB sites as in the resident
// kernel.  Bound by its loads: 256 lattices of
// 32^3 take 8 us (site by site 129).
template <int MODEL, int NB>
__global__ void __launch_bounds__(256) k_plane_stats(TriArgs a, int rec_row) {
    constexpr bool TRI = MODEL == kModelIsingTri;
    const int r = blockIdx.y;
    const RepDev D = a.reps[r];
    const int Lx = D.Lx, Ly = D.Ly, Lz = TRI ? 1 : D.q;
    const uint32_t psz = (uint32_t)(Lx * Ly * Lz / (TRI ? 3 : 2));
    const int items = (int)(psz / (4 * NB));
    const int8_t* lat = a.lat + D.lat_off;
    int cnt[4] = {0, 0, 0, 0}, n = 0;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < items; i += gridDim.x * blockDim.x) {
        // spins +-1 as bytes 01 and FF
        count_item<MODEL, NB, 0x02020202u>(lat, psz, plane_item<MODEL, NB>(i, Lx, Ly, Lz), Ly, Lz,
                                           cnt);
        n += (TRI ? 12 : 8) * NB;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool has = TRI || k < 2 || (k == 2 ? Ly > 1 : Lz > 1);
        cnt[k] = has ? n - 2 * cnt[k] : 0;
    }
    add_sums(cnt, &a.stats[((size_t)rec_row * a.R + r) * a.width]);
}

// Four sites of one Philox block: own bytes S, neighbour counts N (-1
// neighbours per byte); lt holds T - 1 by n + 8 [s = -1] (W < T as a 32-bit
// compare), zero the bits of the entries with T = 0, which never accept.
__device__ __forceinline__ uint32_t plane_decide(uint32_t S, uint32_t N, const uint32_t (&w)[4],
                                                 const uint32_t* lt, uint32_t zero) {
    const uint32_t K = (S << 3) + N, K4 = K << 2;
    const uint8_t* tb = reinterpret_cast<const uint8_t*>(lt);
    uint32_t F = 0u;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        F |= w[u] <= *reinterpret_cast<const uint32_t*>(tb + ((K4 >> (8 * u)) & 0xFFu)) ? 1u << (8 * u)
                                                                                        : 0u;
    if (zero != 0u) {  // uniform over the workgroup
        uint32_t k = K;
        asm volatile("" : "+v"(k));  // keeps this out of the common path
        for (int u = 0; u < 4; ++u)
            if ((zero >> ((k >> (8 * u)) & 15u)) & 1u) F &= ~(1u << (8 * u));
    }
    return S ^ F;
}

// re > 0: after sweep sw0 + sw + 1 = k re of the call the statistics of the
// lattice go to stats row k - 1 (columns 0..3; the caller zeroes the rows).
// They are counts of unequal bonds (and of -1 spins) from the planes, four
// sites a word.  The counts of the launch's rows gather in LDS behind the
// lattice and are stored once at its end, so no sweep waits for global
// memory.
template <int MODEL, int NB, int NI>
__global__ void __launch_bounds__(1024) k_plane_resident(TriArgs a, int n_sweeps, int sw0, int re) {
    extern __shared__ __align__(16) int8_t ls[];
    __shared__ uint32_t lt[16];
    __shared__ uint32_t lzero;
    constexpr bool TRI = MODEL == kModelIsingTri;
    constexpr int ncol = TRI ? 3 : 2;
    const int r = blockIdx.x, tid = (int)threadIdx.x, nthr = (int)blockDim.x;
    const RepDev D = a.reps[r];
    const int Lx = D.Lx, Ly = D.Ly, Lz = TRI ? 1 : D.q;
    const int n = Lx * Ly * Lz;
    const uint32_t psz = (uint32_t)(n / ncol);
    uint32_t* lat = reinterpret_cast<uint32_t*>(a.lat + D.lat_off);
    if (tid == 0) lzero = 0u;
    __syncthreads();
    if (tid < 16) {
        const int k = TRI ? 6 : 2 + 2 * (Ly > 1) + 2 * (Lz > 1);
        const uint64_t T = keyed_threshold(a.tab + (size_t)r * kTriClasses, tid, k);
        lt[tid] = (uint32_t)(T - 1u);
        if (T == 0u && (tid & 7) <= k) atomicOr(&lzero, 1u << tid);
    }
    for (int i = tid; i < n / 4; i += nthr)
        reinterpret_cast<uint32_t*>(ls)[i] = (lat[i] >> 1) & 0x01010101u;
    // recorded rows rec0 .. rec0 + n_rows - 1 (1-based) of this launch
    int* lrec = reinterpret_cast<int*>(ls + ((n + 15) & ~15));
    const int rec0 = re > 0 ? sw0 / re + 1 : 0;
    const int n_rows = re > 0 ? (sw0 + n_sweeps) / re - sw0 / re : 0;
    for (int i = tid; i < 4 * n_rows; i += nthr) lrec[i] = 0;
    const int items = (int)(psz / (4 * NB));
    PlaneItem it0;
    PackedItem itp[NI];
#pragma unroll
    for (int k = 0; k < NI; ++k) {
        it0 = plane_item<MODEL, NB>(min(tid + k * nthr, items - 1), Lx, Ly, Lz);
        itp[k] = pack_item(it0);
    }
    __syncthreads();
    const uint32_t zero = __builtin_amdgcn_readfirstlane(lzero);
    const uint64_t t0 = *a.t_base;
    int next = re > 0 ? rec0 * re - sw0 : 0;  // sweeps to the next recorded one
    for (int sw = 0; sw < n_sweeps; ++sw) {
        const uint64_t t = t0 + (uint64_t)sw;
        for (int c = 0; c < ncol; ++c) {
            const uint32_t p = (uint32_t)((uint64_t)ncol * t + (uint64_t)c);
#pragma unroll
            for (int k = 0; k < NI; ++k) {
                const int i = tid + k * nthr;
                if (i >= items) break;
                const PlaneItem q = NI == 1 ? it0 : unpack_item(itp[k]);
                Words<NB> S, N;
                int8_t* own = ls + (uint32_t)c * psz;
                if (TRI) {
                    const TriWords<NB> w = tri_words<NB, true>(ls, psz, c, q);
                    S = w.S;
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        N.v[b] = w.sa.v[b] + w.fb.v[b] + w.sc.v[b] + w.sd.v[b] + w.fe.v[b] + w.sf.v[b];
                } else {
                    const int8_t* oth = ls + (uint32_t)(1 - c) * psz;
                    Words<NB> M, H;
                    hc_words<NB>(oth, c, q, M, H);
                    S = ldw<NB>(own + q.off);
#pragma unroll
                    for (int b = 0; b < NB; ++b) N.v[b] = M.v[b] + H.v[b];
                    if (Ly > 1) {
                        const Words<NB> u = ldw<NB>(oth + q.ou), d = ldw<NB>(oth + q.od);
#pragma unroll
                        for (int b = 0; b < NB; ++b) N.v[b] += u.v[b] + d.v[b];
                    }
                    if (Lz > 1) {
                        const Words<NB> u = ldw<NB>(oth + q.ozu), d = ldw<NB>(oth + q.ozd);
#pragma unroll
                        for (int b = 0; b < NB; ++b) N.v[b] += u.v[b] + d.v[b];
                    }
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    uint32_t w[4];
                    philox4x32_10((uint32_t)(NB * i + b), p, D.rid, kTriTagMain, a.key0, a.key1, w);
                    S.v[b] = plane_decide(S.v[b], N.v[b], w, lt, zero);
                }
                stw<NB>(own + q.off, S);
            }
            __syncthreads();
        }
        if (re > 0 && sw + 1 == next) {
            int cnt[4] = {0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < NI; ++k) {
                if (tid + k * nthr >= items) break;
                const PlaneItem q = NI == 1 ? it0 : unpack_item(itp[k]);
                count_item<MODEL, NB, ~0u>(ls, psz, q, Ly, Lz, cnt);
            }
            // wave sums (every wave is full and has reconverged)
            int* row = lrec + 4 * ((sw0 + sw + 1) / re - rec0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                cnt[j] = __ockl_wfred_add_i32(cnt[j]);
                if ((tid & 63) == 0) atomicAdd(&row[j], cnt[j]);
            }
            next += re;
            __syncthreads();  // the next sweep writes the lattice
        }
    }
    // counts to sums: n - 2 x (-1 spins, unequal bonds); 0 for an absent dimension
    for (int i = tid; i < 4 * n_rows; i += nthr) {
        const int j = i & 3;
        const bool has = TRI || j < 2 || (j == 2 ? Ly > 1 : Lz > 1);
        a.stats[((size_t)(rec0 - 1 + (i >> 2)) * a.R + r) * a.width + j] = has ? n - 2 * lrec[i] : 0;
    }
    for (int i = tid; i < n / 4; i += nthr)
        lat[i] = reinterpret_cast<const uint32_t*>(ls)[i] * 0xFEu + 0x01010101u;
}

// The same launch for every other width (a plane row of W >= 4 sites): a Philox
// block's four sites may run on into the next row, so a lane works site by site,
// on the lattice in natural order -- a site's partners are then at the same
// distances in every colour, but for the wraps, which depend on the row (worked out
// for the block's two rows) and on x.  The statistics of a recorded sweep come from
// its passes: a bond is counted with its later end, whose partner is final.
// About 270 lane-instructions a block, 60 of them Philox, which bound a full chip:
// 512 triangular 75^2 take 6.4 us a sweep and 7.9 a recorded one (streamed 19.4 and
// 35.1), 256 x 30^3 14.7 and 16.0 (34.0 and 89.0).
namespace {
struct RowAt {
    int base, up, dn, zu, zd;  // row's first site; from a site to its partners in y and z
    int ph;                    // x of the colour's first site
};

template <int MODEL>
__device__ __forceinline__ RowAt row_at(int row, int c, int Lx, int Ly, int Lz, uint32_t mY) {
    RowAt r;
    const int z = MODEL == kModelIsingTri || Lz == 1 ? 0 : (Ly == 1 ? row : (int)__umulhi((uint32_t)row, mY));
    const int y = row - z * Ly, slab = Lx * Ly;
    r.base = row * Lx;
    r.up = y == 0 ? slab - Lx : -Lx;
    r.dn = y + 1 == Ly ? Lx - slab : Lx;
    r.zu = z == 0 ? slab * (Lz - 1) : -slab;
    r.zd = z + 1 == Lz ? slab * (1 - Lz) : slab;
    r.ph = MODEL == kModelIsingTri ? (c + y) % 3 : (c + y + z) & 1;
    return r;
}
}  // namespace

template <int MODEL>
__global__ void __launch_bounds__(1024) k_plane_resident_any(TriArgs a, int n_sweeps, int sw0,
                                                             int re) {
    extern __shared__ __align__(16) uint8_t lsn[];  // a spin a byte (1 for -1) | recorded rows
    __shared__ uint32_t lt[16];
    __shared__ uint32_t lzero;
    constexpr bool TRI = MODEL == kModelIsingTri;
    constexpr int ncol = TRI ? 3 : 2;
    const int r = blockIdx.x, tid = (int)threadIdx.x, nthr = (int)blockDim.x;
    const RepDev D = a.reps[r];
    const int Lx = D.Lx, Ly = D.Ly, Lz = TRI ? 1 : D.q, W = Lx / ncol, rows = Ly * Lz;
    const int n = Lx * rows, nk = n / ncol;
    const bool hy = TRI || Ly > 1, hz = !TRI && Lz > 1;
    // exact quotients b / d for b d < 2^32, d > 1
    const uint32_t mW = 0xFFFFFFFFu / (uint32_t)W + 1u, mY = 0xFFFFFFFFu / (uint32_t)Ly + 1u;
    int8_t* lat = a.lat + D.lat_off;
    if (tid == 0) lzero = 0u;
    __syncthreads();
    if (tid < 16) {
        const int k = TRI ? 6 : 2 + 2 * (Ly > 1) + 2 * (Lz > 1);
        const uint64_t T = keyed_threshold(a.tab + (size_t)r * kTriClasses, tid, k);
        lt[tid] = (uint32_t)(T - 1u);
        if (T == 0u && (tid & 7) <= k) atomicOr(&lzero, 1u << tid);
    }
    // place in natural order of site k of colour c
    const auto place = [&](int c, int k) {
        const int row = (int)__umulhi((uint32_t)k, mW);
        return row * Lx + ncol * (k - row * W) + row_at<MODEL>(row, c, Lx, Ly, Lz, mY).ph;
    };
    for (int c = 0; c < ncol; ++c)
#pragma unroll 4
        for (int k = tid; k < nk; k += nthr) lsn[place(c, k)] = ((uint8_t)lat[c * nk + k] >> 1) & 1u;
    int* lrec = reinterpret_cast<int*>(lsn + ((n + 15) & ~15));
    const int rec0 = re > 0 ? sw0 / re + 1 : 0;
    const int n_rows = re > 0 ? (sw0 + n_sweeps) / re - sw0 / re : 0;
    for (int i = tid; i < 4 * n_rows; i += nthr) lrec[i] = 0;
    __syncthreads();
    const uint32_t zero = __builtin_amdgcn_readfirstlane(lzero);
    const uint64_t t0 = *a.t_base;
    int next = re > 0 ? rec0 * re - sw0 : 0;  // sweeps to the next recorded one
    for (int sw = 0; sw < n_sweeps; ++sw) {
        const bool rec = re > 0 && sw + 1 == next;
        int cnt[4] = {0, 0, 0, 0};
        for (int c = 0; c < ncol; ++c) {
            const uint32_t p = (uint32_t)((uint64_t)ncol * (t0 + (uint64_t)sw) + (uint64_t)c);
            for (int b = tid; 4 * b < nk; b += nthr) {
                const int row = (int)__umulhi((uint32_t)(4 * b), mW), j0 = 4 * b - row * W;
                const RowAt ra = row_at<MODEL>(row, c, Lx, Ly, Lz, mY);
                const RowAt rb = row_at<MODEL>(min(row + 1, rows - 1), c, Lx, Ly, Lz, mY);
                int at[4], s[4], N[4], nx[4], ny[4], nz[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bool nr = j0 + u >= W;  // in the block's second row
                    const int x = ncol * (nr ? j0 + u - W : j0 + u) + (nr ? rb.ph : ra.ph);
                    const int o = (nr ? rb.base : ra.base) + x;
                    const int ol = x == 0 ? o + Lx - 1 : o - 1, orr = x + 1 == Lx ? o + 1 - Lx : o + 1;
                    at[u] = o;
                    s[u] = lsn[o];
                    if (TRI) {
                        // nx the partners of the next colour, ny those of the one before
                        const int up = nr ? rb.up : ra.up, dn = nr ? rb.dn : ra.dn;
                        const int l = lsn[ol], d = lsn[o + dn], ur = lsn[orr + up];
                        const int R = lsn[orr], U = lsn[o + up], dl = lsn[ol + dn];
                        N[u] = l + d + ur + R + U + dl;
                        // by colour: c - 1 (bit fields l, d, ur), all (sums by direction)
                        nx[u] = l | (d << 8) | (ur << 16);
                        ny[u] = (l + R) | ((d + U) << 8) | ((ur + dl) << 16);
                    } else {
                        nx[u] = lsn[ol] + lsn[orr];
                        ny[u] = nz[u] = 0;
                        if (hy) ny[u] = lsn[o + (nr ? rb.up : ra.up)] + lsn[o + (nr ? rb.dn : ra.dn)];
                        if (hz) nz[u] = lsn[o + (nr ? rb.zu : ra.zu)] + lsn[o + (nr ? rb.zd : ra.zd)];
                        N[u] = nx[u] + ny[u] + nz[u];
                    }
                }
                uint32_t w[4];
                philox4x32_10((uint32_t)b, p, D.rid, kTriTagMain, a.key0, a.key1, w);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int K = N[u] + 8 * s[u];
                    const bool in = 4 * b + u < nk;
                    bool f = w[u] <= lt[K];
                    if (zero != 0u) f = f && ((zero >> K) & 1u) == 0u;  // uniform
                    s[u] ^= f ? 1 : 0;
                    if (in) lsn[at[u]] = (uint8_t)s[u];
                    if (rec && in) {  // rec uniform
                        cnt[0] += s[u];
                        if (TRI) {
                            // unequal bonds of a -1 spin: partners less those of -1
                            const int m = c == 0 ? 0 : (c == 1 ? nx[u] : ny[u]);
                            const int full = c == 0 ? 0 : (c == 1 ? 0x010101 : 0x020202);
                            const int e = s[u] ? full - m : m;
                            cnt[1] += e & 0xFF;
                            cnt[2] += (e >> 8) & 0xFF;
                            cnt[3] += e >> 16;
                        } else if (c == 1) {
                            cnt[1] += s[u] ? 2 - nx[u] : nx[u];
                            cnt[2] += s[u] ? 2 - ny[u] : ny[u];
                            cnt[3] += s[u] ? 2 - nz[u] : nz[u];
                        }
                    }
                }
            }
            __syncthreads();
        }
        if (rec) {
            int* row = lrec + 4 * ((sw0 + sw + 1) / re - rec0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                cnt[j] = __ockl_wfred_add_i32(cnt[j]);
                if ((tid & 63) == 0) atomicAdd(&row[j], cnt[j]);
            }
            next += re;
        }
    }
    __syncthreads();
    // counts to sums: n - 2 x (-1 spins, unequal bonds); 0 for an absent dimension
    for (int i = tid; i < 4 * n_rows; i += nthr) {
        const int j = i & 3;
        const bool has = j < 2 || (j == 2 ? hy : TRI || hz);
        a.stats[((size_t)(rec0 - 1 + (i >> 2)) * a.R + r) * a.width + j] = has ? n - 2 * lrec[i] : 0;
    }
    for (int c = 0; c < ncol; ++c)
#pragma unroll 4
        for (int k = tid; k < nk; k += nthr) lat[c * nk + k] = lsn[place(c, k)] ? (int8_t)-1 : (int8_t)1;
}

namespace {
const void* plane_resident_fn(bool hc, int nb, int ni) {
    if (hc)
        return nb == 2 ? (ni == 1 ? (const void*)k_plane_resident<kModelIsingHC, 2, 1>
                                  : (const void*)k_plane_resident<kModelIsingHC, 2, 4>)
                       : (ni == 1 ? (const void*)k_plane_resident<kModelIsingHC, 1, 1>
                                  : (const void*)k_plane_resident<kModelIsingHC, 1, 8>);
    return nb == 2 ? (ni == 1 ? (const void*)k_plane_resident<kModelIsingTri, 2, 1>
                              : (const void*)k_plane_resident<kModelIsingTri, 2, 4>)
                   : (ni == 1 ? (const void*)k_plane_resident<kModelIsingTri, 1, 1>
                              : (const void*)k_plane_resident<kModelIsingTri, 1, 8>);
}
}  // namespace

hipError_t launch_plane_resident(const TriArgs& a, int n_sweeps, int sw0, int re, int lds_bytes,
                                 hipStream_t s) {
    const bool hc = a.model == kModelIsingHC;
    if (!(hc ? a.all_lx8 : a.all_lx12)) {
        const void* fn = hc ? (const void*)k_plane_resident_any<kModelIsingHC>
                            : (const void*)k_plane_resident_any<kModelIsingTri>;
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
        TriArgs b = a;
        void* args[] = {&b, &n_sweeps, &sw0, &re};
        return hipLaunchKernel(fn, dim3(a.R), dim3(std::min(1024, (a.max_blocks + 63) & ~63)), args,
                               lds_bytes, s);
    }
    // one block a lane where the lanes suffice (more waves, shorter chains: 512
    // sites 0.54 us a sweep against 1.13, 1024 triangular 96 x 96 lattices 4.9
    // against 6.0), else two, which share half their reads (256 lattices of
    // 128 x 128: 2.2 us against 2.7)
    const int nb = a.even_blocks && a.max_blocks > 1024 ? 2 : 1;
    const int items = (a.max_blocks + nb - 1) / nb;
    const int ni = (items + 1023) / 1024;
    if (ni > 8 / nb) return hipErrorInvalidValue;  // lattices above 64 KiB
    const int threads = ((items + ni - 1) / ni + 63) & ~63;
    const void* fn = plane_resident_fn(hc, nb, ni);
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (e != hipSuccess) return e;
    TriArgs b = a;
    void* args[] = {&b, &n_sweeps, &sw0, &re};
    return hipLaunchKernel(fn, dim3(a.R), dim3(threads), args, lds_bytes, s);
}

hipError_t launch_tri_init(const TriArgs& a, hipStream_t s) {
    const int nb = (a.max_sites + 3) / 4;
    hipLaunchKernelGGL(k_tri_init, dim3((nb + 255) / 256, a.R), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_tri_pass(const TriArgs& a, int c, int sweep_off, hipStream_t s) {
    // two blocks per lane from 1 M blocks per pass (two for every lane the
    // chip holds at once) when a replica has at least 2048 (four workgroups of
    // 512 blocks: little lost to a ragged last one)
    const bool two = (int64_t)a.max_blocks * a.R >= (int64_t)1 << 20 && a.max_blocks >= 2048;
    const int gx1 = (a.max_blocks + 255) / 256, gx2 = (a.max_blocks + 511) / 512;
    const dim3 g1((unsigned)gx1 * a.R), g2((unsigned)gx2 * a.R);
    if (a.model == kModelIsingHC && a.all_lx8) {
        if (two)
            hipLaunchKernelGGL(k_hc_pass4<2>, g2, dim3(256), 0, s, a, c, sweep_off, gx2);
        else
            hipLaunchKernelGGL(k_hc_pass4<1>, g1, dim3(256), 0, s, a, c, sweep_off, gx1);
    } else if (a.model == kModelIsingHC)
        hipLaunchKernelGGL(k_plane_pass_any<kModelIsingHC>, dim3((a.max_blocks + 255) / 256, a.R), dim3(256), 0, s, a,
                           c, sweep_off);
    else if (a.all_lx12 && two)
        hipLaunchKernelGGL(k_tri_pass4<2>, g2, dim3(256), 0, s, a, c, sweep_off, gx2);
    else if (a.all_lx12)
        hipLaunchKernelGGL(k_tri_pass4<1>, g1, dim3(256), 0, s, a, c, sweep_off, gx1);
    else
        hipLaunchKernelGGL(k_plane_pass_any<kModelIsingTri>, dim3((a.max_blocks + 255) / 256, a.R), dim3(256), 0, s, a,
                           c, sweep_off);
    return hipGetLastError();
}

hipError_t launch_tri_stats(const TriArgs& a, int rec_row, hipStream_t s) {
    const int per = (a.max_sites + 255) / 256;
    const bool hc = a.model == kModelIsingHC;
    if (hc ? a.all_lx8 : a.all_lx12) {
        // four items a lane, as many workgroups as that gives up to 64 a lattice
        const int nb = a.even_blocks ? 2 : 1;
        const int gx = std::min(64, (a.max_blocks / nb + 1023) / 1024);
        const dim3 g(gx, a.R), b(256);
        if (hc && nb == 2)
            hipLaunchKernelGGL((k_plane_stats<kModelIsingHC, 2>), g, b, 0, s, a, rec_row);
        else if (hc)
            hipLaunchKernelGGL((k_plane_stats<kModelIsingHC, 1>), g, b, 0, s, a, rec_row);
        else if (nb == 2)
            hipLaunchKernelGGL((k_plane_stats<kModelIsingTri, 2>), g, b, 0, s, a, rec_row);
        else
            hipLaunchKernelGGL((k_plane_stats<kModelIsingTri, 1>), g, b, 0, s, a, rec_row);
    } else if (hc)
        hipLaunchKernelGGL(k_plane_stats_any<kModelIsingHC>, dim3(std::min(64, (per + 7) / 8), a.R),
                           dim3(256), 0, s, a, rec_row);
    else
        hipLaunchKernelGGL(k_plane_stats_any<kModelIsingTri>, dim3(std::min(64, (per + 7) / 8), a.R),
                           dim3(256), 0, s, a, rec_row);
    return hipGetLastError();
}

hipError_t launch_tri_observables(const TriArgs& a, double* obs, hipStream_t s) {
    hipLaunchKernelGGL(k_tri_observables, dim3((a.R + 127) / 128), dim3(128), 0, s, a, obs);
    return hipGetLastError();
}

}  // namespace spinmc
