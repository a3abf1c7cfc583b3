// Multispin-coded square-lattice Ising (1-bit spins): 32 replicas with the
// same lattice shape, couplings, field and temperature packed bit by bit in
// one uint32 per site (bit b = 1 is s = +1 in replica b).  On the device a
// group's words sit in two colour planes, as the byte planes of the square
// lattice: site (y, x) is word (y, x >> 1) of plane (x + y) & 1, each plane
// Ly rows of W = Lx / 2 words.  The replicas share the random numbers, so
// one Philox word decides 32 attempts: in pass p = 2t + c (colour
// c = (x + y) & 1) the site with within-colour index k = (y Lx + x) >> 1 --
// its plane word index y W + (x >> 1) -- takes W = word k & 3 of block
// (k >> 2, p, rid, 0), and every bit whose class idx = 9 [s > 0] +
// 3 (Sx/2 + 1) + (Sy/2 + 1) has W < T[idx] flips (Algorithm 1; the
// thresholds are the FP64 host table of the square lattice).  The classes of
// all 32 bits come from bitwise logic: a neighbour bit agrees with the own
// bit where their xor is 0, and counts of 0, 1 or 2 agreeing horizontal
// (vertical) neighbours are ~(a | b), a ^ b and a & b.
//
// Lx is a multiple of 8: a lane takes the four sites of one Philox block,
// four consecutive words of a row of plane c, and reads the other plane's
// same row (its horizontal neighbours, with one halo word on the side of the
// row parity) and rows y - 1, y + 1 (vertical neighbours) as 16-byte loads;
// only the own plane is written.
#include "msc_internal.hpp"

namespace spinmc {

namespace {
constexpr uint32_t kMscTagMain = 0u, kMscTagInit = 2u;

__device__ __forceinline__ uint32_t e4(const uint4& v, int i) {
    return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w));
}

// Word index of site (y, x) of a group's lattice in its colour planes.
__device__ __forceinline__ size_t plane_word(int y, int x, int Lx, int Ly) {
    const int W = Lx >> 1;
    return (size_t)((x + y) & 1) * Ly * W + (size_t)y * W + (x >> 1);
}
}  // namespace

// Bit b of site n: 1 iff word n & 3 of block (n >> 2, b, rid, 2) is < 2^31.
__global__ void __launch_bounds__(256) k_msc_init(MscArgs a) {
    const RepDev D = a.reps[blockIdx.y];
    const int n = D.Lx * D.Ly;
    const int q = blockIdx.x * blockDim.x + threadIdx.x;  // block of 4 sites
    if (4 * q >= n) return;
    uint32_t v[4] = {0u, 0u, 0u, 0u};
    for (int b = 0; b < 32; ++b) {
        uint32_t w[4];
        philox4x32_10((uint32_t)q, (uint32_t)b, D.rid, kMscTagInit, a.key0, a.key1, w);
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] |= (w[u] < 0x80000000u ? 1u : 0u) << b;
    }
    uint32_t* lat = reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(a.lat) + D.lat_off);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int i = 4 * q + u;
        if (i < n) {
            const int y = i / D.Lx;
            lat[plane_word(y, i - y * D.Lx, D.Lx, D.Ly)] = v[u];
        }
    }
}

// ------------------------------------------------------------ flip rule
// What a group's thresholds have in common decides how much logic a word
// needs (msc_mode on the host):
//   ISO  (h = 0, Jx = Jy): a bit's class is its number n of agreeing
//        neighbours; three of the five always flip and two are compared, n = 4
//        and 3 (inv = 0), or n = 0 and 1 (inv = ~0, both couplings negative:
//        the same rule on the complemented own bit)
//   SYM  (h = 0): the class of -1 is that of +1 counted by agreement, nine
//        compares
//   ANY  eighteen compares, one set for each spin value
// Operations a word beyond its quarter of a Philox block (14 lane-cycles):
// 12 + 4, ~40 and ~70; the rule of eighteen for all was ~90.
struct IsoRule {
    uint32_t t3, t4, inv;
    __device__ __forceinline__ void load(const uint64_t* tg) {
        inv = tg[9 + 8] == (1ull << 32) ? ~0u : 0u;  // n = 4 always flips
        t4 = (uint32_t)(inv ? tg[9] : tg[9 + 8]);
        t3 = (uint32_t)(inv ? tg[9 + 1] : tg[9 + 7]);
    }
    __device__ __forceinline__ uint32_t flip(uint32_t s, uint32_t l, uint32_t r, uint32_t u,
                                             uint32_t d, uint32_t W) const {
        const uint32_t o = s ^ inv;
        const uint32_t x2 = ~(o ^ l) & ~(o ^ r), y2 = ~(o ^ u) & ~(o ^ d);
        const uint32_t x1 = l ^ r, y1 = u ^ d;
        const uint32_t n4 = ~(x2 & y2);
        const uint32_t n3 = ~((x1 & y2) | (x2 & y1));
        return (W < t3 ? ~0u : n3) & (W < t4 ? ~0u : n4);
    }
};

// One of 3 x 3 compare masks by the one-hot pairs (x1, x2), (y1, y2).
__device__ __forceinline__ uint32_t sel9(const uint32_t* m, uint32_t x1, uint32_t x2, uint32_t y1,
                                         uint32_t y2) {
    uint32_t g[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const uint32_t t = (m[3 * i + 1] & y1) | (m[3 * i] & ~y1);
        g[i] = (m[3 * i + 2] & y2) | (t & ~y2);
    }
    const uint32_t t = (g[1] & x1) | (g[0] & ~x1);
    return (g[2] & x2) | (t & ~x2);
}

// W < T as a 32-bit compare: W <= T - 1 for 1 <= T <= 2^32, and never for
// T = 0 (uniform per class: scalar registers and scalar logic).
template <int N>
struct CmpRule {
    uint32_t tm1[N];
    bool never[N];
    __device__ __forceinline__ void load(const uint64_t* tg) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint64_t T = tg[kMscClasses - N + i];
            never[i] = T == 0;
            tm1[i] = T == 0 ? 0u : (uint32_t)(T - 1);
        }
    }
    __device__ __forceinline__ uint32_t flip(uint32_t s, uint32_t l, uint32_t r, uint32_t u,
                                             uint32_t d, uint32_t W) const {
        uint32_t m[N];
#pragma unroll
        for (int i = 0; i < N; ++i) m[i] = (W <= tm1[i] && !never[i]) ? ~0u : 0u;
        const uint32_t x1 = l ^ r, y1 = u ^ d;
        if constexpr (N == 9) {  // agreement counts
            return sel9(m, x1, ~(s ^ l) & ~(s ^ r), y1, ~(s ^ u) & ~(s ^ d));
        } else {  // counts of +1
            const uint32_t x2 = l & r, y2 = u & d;
            const uint32_t fn = sel9(m, x1, x2, y1, y2), fp = sel9(m + 9, x1, x2, y1, y2);
            return (s & fp) | (~s & fn);
        }
    }
};

template <int MODE>
struct RuleOf {
    using T = CmpRule<MODE == kMscSym ? 9 : 18>;
};
template <>
struct RuleOf<kMscIso> {
    using T = IsoRule;
};

// Four words of a row: the own words S, the other plane's same row M with
// its halo word on side par (own site of word j: x = 2 j + par), rows above
// and below.
template <class RULE>
__device__ __forceinline__ uint4 update4(const RULE& f, const uint4& S, const uint4& M,
                                         uint32_t halo, bool par, const uint4& U, const uint4& D,
                                         const uint32_t* w) {
    uint32_t nv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        // left (x - 1) and right (x + 1) neighbours: words j - 1 + par and j + par
        const uint32_t l = par ? e4(M, u) : (u == 0 ? halo : e4(M, u - 1));
        const uint32_t r = par ? (u == 3 ? halo : e4(M, u + 1)) : e4(M, u);
        const uint32_t s = e4(S, u);
        nv[u] = s ^ f.flip(s, l, r, e4(U, u), e4(D, u), w[u]);
    }
    return make_uint4(nv[0], nv[1], nv[2], nv[3]);
}

// ------------------------------------------------------------- bit counts
__device__ __forceinline__ uint32_t maj(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xe8);
}

// Thirty-two counts at once, one a replica, as bit planes: bit b of p[k] is
// bit k of replica b's count.
template <int P>
struct BitCount {
    uint32_t p[P];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int k = 0; k < P; ++k) p[k] = 0u;
    }
    // adds the Q-plane counts q
    template <int Q>
    __device__ __forceinline__ void add(const uint32_t (&q)[Q]) {
        uint32_t c = p[0] & q[0];
        p[0] ^= q[0];
#pragma unroll
        for (int k = 1; k < P; ++k) {
            const uint32_t o = p[k];
            if (k < Q) {
                p[k] = xor3(o, q[k], c);
                c = maj(o, q[k], c);
            } else {
                p[k] = o ^ c;
                c &= o;
            }
        }
    }
    // adds eight words of one bit a replica
    __device__ __forceinline__ void add8(const uint32_t (&v)[8]) {
        uint32_t s0, s1, s2, c0, c1, c2, c3, t, q[4];
        auto fa = [](uint32_t a, uint32_t b, uint32_t c, uint32_t& sum, uint32_t& car) {
            sum = xor3(a, b, c);
            car = maj(a, b, c);
        };
        fa(v[0], v[1], v[2], s0, c0);
        fa(v[3], v[4], v[5], s1, c1);
        fa(s0, s1, v[6], s2, c2);
        q[0] = s2 ^ v[7];
        c3 = s2 & v[7];
        uint32_t d0, d1;
        fa(c0, c1, c2, t, d0);
        q[1] = t ^ c3;
        d1 = t & c3;
        q[2] = d0 ^ d1;
        q[3] = d0 & d1;
        add(q);
    }
};

// The value of another lane: in steps 0 .. 3 one of the other half of a group
// of 2, 4, 8, 16 lanes whose halves each agree, by data-parallel-primitive
// moves; in steps 4 and 5 lane ^ 16 and lane ^ 32.
template <int STEP>
__device__ __forceinline__ uint32_t other_half(uint32_t v) {
    // quad_perm 1 0 3 2, quad_perm 2 3 0 1, row_half_mirror, row_mirror
    constexpr int kCtrl[4] = {0xB1, 0x4E, 0x141, 0x140};
    if constexpr (STEP < 4)
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl[STEP], 0xf, 0xf, true);
    else
        return (uint32_t)__shfl_xor((int)v, 1 << STEP, 64);
}

template <int STEP, int P, int N>
__device__ __forceinline__ void wave_steps(BitCount<N> (&a)[3]) {
    if constexpr (STEP < 6) {
        uint32_t q[3][P + STEP];
#pragma unroll
        for (int m = 0; m < 3; ++m)
#pragma unroll
            for (int k = 0; k < P + STEP; ++k) q[m][k] = other_half<STEP>(a[m].p[k]);
#pragma unroll
        for (int m = 0; m < 3; ++m) a[m].add(q[m]);
        wave_steps<STEP + 1, P>(a);
    }
}

// Adds the three counts of a wave's 64 lanes (each below 2^P) to cnt[3][32] in
// LDS.
template <int P>
__device__ __forceinline__ void wave_count(const BitCount<P> (&v)[3], int* cnt) {
    BitCount<P + 6> a[3];
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
        for (int k = 0; k < P + 6; ++k) a[m].p[k] = k < P ? v[m].p[k] : 0u;
    wave_steps<0, P>(a);
    const int lane = threadIdx.x & 63;
    if (lane < 32) {
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            int n = 0;
#pragma unroll
            for (int k = 0; k < P + 6; ++k) n |= (int)((a[m].p[k] >> lane) & 1u) << k;
            atomicAdd(&cnt[32 * m + lane], n);
        }
    }
}

// Row r's bits of a colour-1 quad: S own words, N the other plane's same row
// with its halo; every bond joins the colours, so the bonds of the colour-1
// sites are all bonds.
template <int P>
__device__ __forceinline__ void count_row(BitCount<P> (&ct)[3], const uint4& S, const uint4& M,
                                          uint32_t halo, bool par, const uint4& U,
                                          const uint4& D) {
    uint32_t v[8];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        v[u] = e4(S, u);
        v[4 + u] = e4(M, u);
    }
    ct[0].add8(v);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t l = par ? e4(M, u) : (u == 0 ? halo : e4(M, u - 1));
        const uint32_t r = par ? (u == 3 ? halo : e4(M, u + 1)) : e4(M, u);
        v[u] = e4(S, u) ^ l;
        v[4 + u] = e4(S, u) ^ r;
    }
    ct[1].add8(v);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        v[u] = e4(S, u) ^ e4(U, u);
        v[4 + u] = e4(S, u) ^ e4(D, u);
    }
    ct[2].add8(v);
}

// --------------------------------------------------------------- streamed
template <int MODE>
__global__ void __launch_bounds__(256) k_msc_pass4(MscArgs a, int c, int sweep_off) {
    const int g = blockIdx.y;
    typename RuleOf<MODE>::T rule;
    rule.load(a.tab + (size_t)g * kMscClasses);
    const RepDev D = a.reps[g];
    const int Lx = D.Lx, Ly = D.Ly, W = Lx >> 1, qpr = W >> 2;
    const int b = blockIdx.x * blockDim.x + threadIdx.x;  // Philox block = word (y W + j0) / 4
    if (b >= Ly * qpr) return;
    const int y = b / qpr, j0 = 4 * (b - y * qpr);
    const int par = (c + y) & 1;  // own site of word j: x = 2 j + par
    const int yu = y == 0 ? Ly - 1 : y - 1, yd = y + 1 == Ly ? 0 : y + 1;
    uint32_t* lat = reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(a.lat) + D.lat_off);
    uint32_t* own = lat + (size_t)c * Ly * W;
    const uint32_t* oth = lat + (size_t)(1 - c) * Ly * W;
    const uint4 S = *reinterpret_cast<const uint4*>(own + (size_t)y * W + j0);
    const uint4 M = *reinterpret_cast<const uint4*>(oth + (size_t)y * W + j0);
    const uint4 U = *reinterpret_cast<const uint4*>(oth + (size_t)yu * W + j0);
    const uint4 Dn = *reinterpret_cast<const uint4*>(oth + (size_t)yd * W + j0);
    // the horizontal neighbour outside the four words: word j0 - 1 (par 0)
    // or j0 + 4 (par 1) of the other plane's row, periodic
    const uint32_t halo =
        oth[(size_t)y * W + (par ? (j0 + 4 == W ? 0 : j0 + 4) : (j0 == 0 ? W - 1 : j0 - 1))];
    const uint64_t t = *a.t_base + (uint64_t)sweep_off;
    const uint32_t p = (uint32_t)(2 * t + (uint64_t)c);
    uint32_t w[4];
    philox4x32_10((uint32_t)b, p, D.rid, kMscTagMain, a.key0, a.key1, w);
    *reinterpret_cast<uint4*>(own + (size_t)y * W + j0) =
        update4(rule, S, M, halo, par, U, Dn, w);
}

// Per bit b: M = 2 ones - N, Bx = N - 2 (ones of s ^ right), By likewise.
// A lane adds up to 15 quads of colour 1 (counts below 128) as bit planes, a
// wave adds its lanes in six steps, one LDS atomic a wave, bit and statistic.
// Bound by its loads: 256 groups of 256 x 256 take 21 us, where ballots of
// every word's 32 bits took 407.
__global__ void __launch_bounds__(256) k_msc_stats(MscArgs a, int rec_row) {
    __shared__ int cnt[3][32];
    const int g = blockIdx.y;
    const RepDev D = a.reps[g];
    const int Lx = D.Lx, Ly = D.Ly, W = Lx >> 1, qpr = W >> 2, nb = Ly * qpr;
    if (threadIdx.x < 96) (&cnt[0][0])[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t* p0 =
        reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(a.lat) + D.lat_off);
    const uint32_t* p1 = p0 + (size_t)Ly * W;
    const int stride = gridDim.x * blockDim.x;
    int visited = 0;  // sites of this workgroup
    for (int base = blockIdx.x * blockDim.x; base < nb;) {
        BitCount<7> ct[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) ct[k].clear();
        for (int it = 0; it < 15 && base < nb; ++it, base += stride) {
            visited += 8 * min((int)blockDim.x, nb - base);
            const int b = base + threadIdx.x;
            if (b >= nb) continue;
            const int y = b / qpr, j0 = 4 * (b - y * qpr);
            const int par = (1 + y) & 1;
            const int yu = y == 0 ? Ly - 1 : y - 1, yd = y + 1 == Ly ? 0 : y + 1;
            const uint4 S = *reinterpret_cast<const uint4*>(p1 + (size_t)y * W + j0);
            const uint4 M = *reinterpret_cast<const uint4*>(p0 + (size_t)y * W + j0);
            const uint4 U = *reinterpret_cast<const uint4*>(p0 + (size_t)yu * W + j0);
            const uint4 Dn = *reinterpret_cast<const uint4*>(p0 + (size_t)yd * W + j0);
            const uint32_t halo = p0[(size_t)y * W + (par ? (j0 + 4 == W ? 0 : j0 + 4)
                                                          : (j0 == 0 ? W - 1 : j0 - 1))];
            count_row(ct, S, M, halo, par, U, Dn);
        }
        wave_count(ct, &cnt[0][0]);
    }
    __syncthreads();
    if (threadIdx.x < 32) {
        const int bit = threadIdx.x;
        int32_t* row = a.stats + ((size_t)rec_row * (32 * a.G) + 32 * g + bit) * a.width;
        // every workgroup adds its share of 2 ones - N as 2 ones - visited
        atomicAdd(&row[0], 2 * cnt[0][bit] - visited);
        atomicAdd(&row[1], visited - 2 * cnt[1][bit]);
        atomicAdd(&row[2], visited - 2 * cnt[2][bit]);
    }
}

// --------------------------------------------------------------- resident
// Whole runs of a group in one workgroup, the lattice in registers: lane
// (q, ch) holds words 4 q .. 4 q + 3 of rows NR ch .. NR ch + NR - 1 of both
// planes (8 NR registers) and sees its neighbours' through LDS -- of each
// plane the lane's first and last row and, of each row, the one edge word
// that a neighbour's update of the other colour reads.  A plane's slots are
// written in its own pass and read in the other's, so one barrier a pass
// orders both.  Bound by its operations (~30 lane-cycles a word in ISO mode,
// half of them Philox): 256 groups of 256 x 256 take 4.8 us a pass, 26.2
// streamed with the rule of eighteen and 19.1 streamed with the ISO rule (9.1 and
// 17 resident against 20.6 and 23.1 with the SYM and ANY rules).
//
// Rows past Ly of the last chunk (NR does not divide Ly) hold copies: they
// are updated like the others, never stored, published or counted.
template <int NR, int MODE>
__global__ void __launch_bounds__(1024) k_msc_resident(MscArgs a, int n_sweeps, int sw0, int re) {
    extern __shared__ uint4 msc_lds[];
    const int g = blockIdx.x, T = blockDim.x;
    // LDS of plane k: T first rows, T last rows, then the edge words of the
    // even rows and of the odd rows, NR / 2 a lane; the counts behind both
    constexpr int kPlane = 2 + (NR + 3) / 4, H = NR / 2;
    struct alignas(4 * H) Edge {
        uint32_t w[H];
    };
    int* cnt = reinterpret_cast<int*>(msc_lds + 2 * kPlane * T);
    typename RuleOf<MODE>::T rule;
    rule.load(a.tab + (size_t)g * kMscClasses);
    const RepDev D = a.reps[g];
    const int Lx = D.Lx, Ly = D.Ly, W = Lx >> 1, qpr = W >> 2;
    const int nch = (Ly + NR - 1) / NR;
    const int tid = threadIdx.x;
    const bool active = tid < qpr * nch;
    const int ch = active ? tid / qpr : 0, q = active ? tid - ch * qpr : 0;
    const int me = ch * qpr + q;
    const int y0 = ch * NR, nr = min(NR, Ly - y0);
    const int left = q == 0 ? me + qpr - 1 : me - 1, right = q + 1 == qpr ? me - q : me + 1;
    const int upl = ch == 0 ? (nch - 1) * qpr + q : me - qpr;
    const int dnl = ch + 1 == nch ? q : me + qpr;
    uint32_t* lat = reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(a.lat) + D.lat_off);
    uint4 V[2][NR];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int r = 0; r < NR; ++r)
            V[k][r] = *reinterpret_cast<const uint4*>(
                lat + ((size_t)k * Ly + min(y0 + r, Ly - 1)) * W + 4 * q);
    auto publish = [&](int k) {  // plane k's first row, last row and edge words
        uint4* f = msc_lds + k * kPlane * T;
        Edge* e = reinterpret_cast<Edge*>(f + 2 * T);
        f[me] = V[k][0];
        uint4 last = V[k][NR - 1];
        if (nr < NR) {
#pragma unroll
            for (int r = 0; r < NR - 1; ++r)
                if (nr == r + 1) last = V[k][r];
        }
        f[T + me] = last;
#pragma unroll
        for (int o = 0; o < 2; ++o) {  // the other colour's halo side at row r: (1 - k + r) & 1
            Edge v;
#pragma unroll
            for (int h = 0; h < H; ++h)
                v.w[h] = ((1 - k + o) & 1) ? V[k][2 * h + o].x : V[k][2 * h + o].w;
            e[o * T + me] = v;
        }
    };
    for (int k = tid; k < 96; k += T) cnt[k] = 0;
    if (active) publish(1);
    __syncthreads();
    const uint64_t t0 = *a.t_base;
    const uint32_t blk0 = (uint32_t)(y0 * qpr + q);
    for (int i = 0; i < n_sweeps; ++i) {
        // pass counter of colour 0 (the counter advances after the launch)
        const uint32_t p0 = (uint32_t)(2 * (t0 + (uint64_t)i));
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (active) {
                const uint4* f = msc_lds + (1 - c) * kPlane * T;
                const Edge* e = reinterpret_cast<const Edge*>(f + 2 * T);
                const uint4 U = f[T + upl], Dn = f[dnl];
                const Edge ed[2] = {e[c ? right : left], e[T + (c ? left : right)]};
                if (nr < NR) {  // the row below the last is the lower neighbour's first
#pragma unroll
                    for (int r = 1; r < NR; ++r)
                        if (nr == r) V[1 - c][r] = Dn;
                }
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    uint32_t w[4];
                    uint32_t bb = blk0 + (uint32_t)(r * qpr);
                    asm volatile("" : "+v"(bb));  // not hoisted: registers
                    philox4x32_10(bb, p0 + (uint32_t)c, D.rid, kMscTagMain,
                                  a.key0, a.key1, w);
                    V[c][r] = update4(rule, V[c][r], V[1 - c][r], ed[r & 1].w[r >> 1], (c + r) & 1,
                                      r == 0 ? U : V[1 - c][r - 1],
                                      r + 1 == NR ? Dn : V[1 - c][r + 1], w);
                    __builtin_amdgcn_sched_barrier(0);
                }
                publish(c);
            }
            if (c == 0) __syncthreads();
        }
        const int done = sw0 + i + 1;
        const bool rec = re > 0 && done % re == 0;
        if (rec) {
            BitCount<7> ct[3];  // at most 8 NR = 64 bits of each a replica
#pragma unroll
            for (int k = 0; k < 3; ++k) ct[k].clear();
            if (active) {
                const uint4* f = msc_lds;
                const Edge* e = reinterpret_cast<const Edge*>(f + 2 * T);
                const uint4 U = f[T + upl], Dn = f[dnl];
                const Edge ed[2] = {e[right], e[T + left]};
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (r < nr)
                        count_row(ct, V[1][r], V[0][r], ed[r & 1].w[r >> 1], (1 + r) & 1, r == 0 ? U : V[0][r - 1],
                                  r + 1 == NR ? Dn : V[0][r + 1]);
            }
            wave_count(ct, cnt);
        }
        __syncthreads();
        if (rec && tid < 32) {  // cleared for the next row, at least two barriers away
            const int N = Lx * Ly;
            int32_t* row =
                a.stats + ((size_t)(done / re - 1) * (32 * a.G) + 32 * g + tid) * a.width;
            row[0] = 2 * cnt[tid] - N;
            row[1] = N - 2 * cnt[32 + tid];
            row[2] = N - 2 * cnt[64 + tid];
            cnt[tid] = cnt[32 + tid] = cnt[64 + tid] = 0;
        }
    }
    if (active)
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int r = 0; r < NR; ++r)
                if (r < nr)
                    *reinterpret_cast<uint4*>(lat + ((size_t)k * Ly + y0 + r) * W + 4 * q) =
                        V[k][r];
}

hipError_t launch_msc_init(const MscArgs& a, hipStream_t s) {
    const int nq = (a.max_sites + 3) / 4;
    hipLaunchKernelGGL(k_msc_init, dim3((nq + 255) / 256, a.G), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_msc_pass(const MscArgs& a, int c, int sweep_off, hipStream_t s) {
    const dim3 grid((a.max_blocks + 255) / 256, a.G), wg(256);
    switch (a.mode) {
        case kMscIso: hipLaunchKernelGGL(k_msc_pass4<kMscIso>, grid, wg, 0, s, a, c, sweep_off); break;
        case kMscSym: hipLaunchKernelGGL(k_msc_pass4<kMscSym>, grid, wg, 0, s, a, c, sweep_off); break;
        default: hipLaunchKernelGGL(k_msc_pass4<kMscAny>, grid, wg, 0, s, a, c, sweep_off);
    }
    return hipGetLastError();
}

hipError_t launch_msc_stats(const MscArgs& a, int rec_row, hipStream_t s) {
    // four quads a lane, as many workgroups as that gives up to 64 a group
    const int per = (a.max_blocks + 1023) / 1024;
    hipLaunchKernelGGL(k_msc_stats, dim3(per < 64 ? per : 64, a.G), dim3(256), 0, s, a, rec_row);
    return hipGetLastError();
}

namespace {
template <int NR, int MODE>
hipError_t msc_resident(const MscArgs& a, int n, int sw0, int re, int lanes, hipStream_t s) {
    const size_t lds = msc_resident_lds(NR, lanes);
    auto* k = k_msc_resident<NR, MODE>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)k,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, dim3(a.G), dim3(lanes), lds, s, a, n, sw0, re);
    return hipGetLastError();
}

template <int NR>
hipError_t msc_resident_mode(const MscArgs& a, int n, int sw0, int re, int lanes, hipStream_t s) {
    switch (a.mode) {
        case kMscIso: return msc_resident<NR, kMscIso>(a, n, sw0, re, lanes, s);
        case kMscSym: return msc_resident<NR, kMscSym>(a, n, sw0, re, lanes, s);
        default: return msc_resident<NR, kMscAny>(a, n, sw0, re, lanes, s);
    }
}
}  // namespace

hipError_t launch_msc_resident(const MscArgs& a, int rows, int lanes, int n_sweeps, int sw0, int re,
                               hipStream_t s) {
    if (rows == 2) return msc_resident_mode<2>(a, n_sweeps, sw0, re, lanes, s);
    if (rows == 4) return msc_resident_mode<4>(a, n_sweeps, sw0, re, lanes, s);
    return msc_resident_mode<8>(a, n_sweeps, sw0, re, lanes, s);
}

}  // namespace spinmc
