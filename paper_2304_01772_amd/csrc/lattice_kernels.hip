// Ising and q-state Potts checkerboard Metropolis kernels for gfx950.
//
// Data layout (per replica): two int8 colour planes P0, P1, each Ly rows of
// W = Lx/2 bytes; site (y, x) lives in P[(x+y)&1][y][x>>1].  Ising stores
// the spin bit u = (s + 1)/2, Potts the label.  A colour pass updates every
// byte of P_c from its own value and four neighbours in P_{1-c}: the same
// column in rows y-1, y, y+1, and column j-1 (if x is even) or j+1 (if x is
// odd) in row y.  Colour-0 sites go first (Related Work, Fig. 1: sites of one
// colour have no interacting neighbour of that colour, so the pass is
// embarrassingly parallel).
//
// The fast ("chunk") path gives each lane 16 consecutive bytes of a plane row
// (one dwordx4 load per plane row), builds neighbour sums with byte-SWAR
// arithmetic, and consumes one 16-bit Philox prefix per site for the
// Metropolis test of Algorithm 1 (Ising: 8 sites per Philox4x32-10 call, two
// sites a lookup and compare;
// Potts: 16-bit proposal + 16-bit accept prefix, 4 sites per call).  The low
// 16 bits of the uniform word are drawn from the fallback stream only when
// the prefix ties the threshold's high half (probability 2^-16), so the
// result equals comparing a full 32-bit uniform word with the FP64-built
// threshold T = ceil(2^32 exp(-beta dE)).
#include "item8.hpp"
#include "spinmc_internal.hpp"

#include <algorithm>

namespace spinmc {

namespace {

__device__ __forceinline__ uint32_t sad_u8(uint32_t a, uint32_t acc) {
    return __builtin_amdgcn_sad_u8(a, 0u, acc);
}

// Wave + workgroup sum of up to 4 ints, result valid in thread 0.
template <int N>
__device__ __forceinline__ void block_sum(int (&v)[N], int* lds /* >= 16*N */) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += __shfl_xor(v[i], o, 64);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nw = (blockDim.x + 63) >> 6;
    __syncthreads();
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) lds[wave * N + i] = v[i];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < nw; ++w) {
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] += lds[w * N + i];
        }
    }
    __syncthreads();
}

struct IsingAcc {
    int M, Bx, By;
};

// 0xFF in byte i where d_i is negative (bit 31 set), else 0: v_perm_b32
// selectors 9 and 11 replicate bit 31 of its low and high source dword,
// 12 gives zero.
__device__ __forceinline__ uint32_t sign_bytes(uint32_t d0, uint32_t d1, uint32_t d2, uint32_t d3) {
    return __builtin_amdgcn_perm(d1, d0, 0x0C0C0B09u) | __builtin_amdgcn_perm(d3, d2, 0x0B090C0Cu);
}

// ---------------------------------------------------------------- Ising
// One 16-site chunk of plane row y starting at byte j0 (j0 % 16 == 0,
// W % 16 == 0): own bytes, the other plane's rows y-1, y, y+1, and the halo
// dword holding the horizontal neighbour of the first (PAR = 0) or last
// (PAR = 1) byte.  Loading is split from computing so that a lane can keep
// two chunks' loads in flight.
// 16-byte accesses of the own-colour plane; NT marks them nontemporal
// (streamed past the caches) for lattice sets larger than the last-level
// cache, where the own plane is read once and written once per pass.
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
template <bool NT>
__device__ __forceinline__ uint4 load_own(const uint8_t* p) {
    if (NT) {
        const u32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
        return make_uint4(t.x, t.y, t.z, t.w);
    }
    return *reinterpret_cast<const uint4*>(p);
}
template <bool NT>
__device__ __forceinline__ void store_own(uint8_t* p, uint32_t a, uint32_t b, uint32_t c,
                                          uint32_t d) {
    if (NT) {
        const u32x4_t t = {a, b, c, d};
        __builtin_nontemporal_store(t, reinterpret_cast<u32x4_t*>(p));
    } else {
        *reinterpret_cast<uint4*>(p) = make_uint4(a, b, c, d);
    }
}

struct ChunkIn {
    uint4 o, m, U, D;
    uint32_t e;
};

// Byte offsets within a plane: oo of the chunk (own row and the other
// plane's same row), uo / dof of the rows above / below, eo of the halo dword.
template <bool NT>
__device__ __forceinline__ ChunkIn chunk_load(const uint8_t* own, const uint8_t* oth, uint32_t oo,
                                              uint32_t uo, uint32_t dof, uint32_t eo) {
    ChunkIn in;
    in.o = load_own<NT>(own + oo);
    in.m = *reinterpret_cast<const uint4*>(oth + oo);
    in.U = *reinterpret_cast<const uint4*>(oth + uo);
    in.D = *reinterpret_cast<const uint4*>(oth + dof);
    in.e = *reinterpret_cast<const uint32_t*>(oth + eo);
    return in;
}

// Plane offsets of one chunk: row offset ro (= y W), column j0; the rows
// above and below wrap periodically, and so does the halo dword.
template <int PAR>
struct ChunkOff {
    uint32_t oo, uo, dof, eo;
    __device__ __forceinline__ ChunkOff(uint32_t ro, uint32_t j0, uint32_t W, uint32_t last) {
        oo = ro + j0;
        uo = (ro == 0u ? last : ro - W) + j0;
        dof = (ro == last ? 0u : ro + W) + j0;
        eo = ro + (PAR == 0 ? (j0 == 0u ? W - 4u : j0 - 4u) : (j0 + 16u == W ? 0u : j0 + 16u));
    }
};

// The shifted byte stream: the horizontal neighbour that the other plane's same
// row does not hold at the own column, left (par 0) or right (par 1).
__device__ __forceinline__ void side_bytes(int par, const uint32_t (&mv)[4], uint32_t e,
                                           uint32_t (&sv)[4]) {
    if (par == 0) {
        sv[0] = __builtin_amdgcn_alignbyte(mv[0], e, 3);
        sv[1] = __builtin_amdgcn_alignbyte(mv[1], mv[0], 3);
        sv[2] = __builtin_amdgcn_alignbyte(mv[2], mv[1], 3);
        sv[3] = __builtin_amdgcn_alignbyte(mv[3], mv[2], 3);
    } else {
        sv[0] = __builtin_amdgcn_alignbyte(mv[1], mv[0], 1);
        sv[1] = __builtin_amdgcn_alignbyte(mv[2], mv[1], 1);
        sv[2] = __builtin_amdgcn_alignbyte(mv[3], mv[2], 1);
        sv[3] = __builtin_amdgcn_alignbyte(e, mv[3], 1);
    }
}

typedef short s16x2_t __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const uint32_t* lds_u32_t;

// Two sites at a time.  The table in LDS holds, for each pair of classes
// (c0, c1), the high halves of both thresholds as signed 16-bit numbers,
// min(T_hi, 65535) - 32768, in one dword: entry 18 c0 + c1, whose byte offset
// 72 c0 + 4 c1 is one byte dot product.  Against the prefixes with their top
// bit flipped one saturating packed subtraction decides both: negative accepts,
// zero is a tie (or T_hi = 65536 at r = 65535) that the exact rule below
// resolves, positive rejects.  The thresholds themselves, [18 hi | 18 lo], lie
// behind the pairs.
constexpr int kIsingPairs = kIsingClasses * kIsingClasses;
static_assert(kIsingTabWords == kIsingPairs + 2 * kIsingClasses, "table layout");

__device__ __forceinline__ void load_ising_table(const uint32_t* tab, const RepDev& R, uint32_t* l,
                                                 int tid, int nthr) {
    const uint32_t* t = tab + R.tab_off;
    for (int i = tid; i < kIsingTabWords; i += nthr) {
        if (i < kIsingPairs) {
            const int c0 = i / kIsingClasses, c1 = i - c0 * kIsingClasses;
            l[i] = (min(t[c0], 65535u) | (min(t[c1], 65535u) << 16)) ^ 0x80008000u;
        } else {
            l[i] = t[i - kIsingPairs];
        }
    }
}

// The ties of an item (bit j of tie: site j), decided by the low halves.
template <int NW>
__device__ __forceinline__ uint32_t ising_ties(uint32_t tie, const uint32_t* tab,
                                               const uint32_t (&idx)[NW], uint32_t kb, uint32_t p,
                                               uint32_t rid, uint32_t k0, uint32_t k1) {
    uint32_t acc = 0u;
    const uint32_t i0 = idx[0], i1 = idx[1], i2 = idx[NW - 2], i3 = idx[NW - 1];
    while (tie != 0u) {
        const uint32_t j = (uint32_t)__builtin_ctz(tie);
        tie &= tie - 1u;
        const uint32_t iw = j < 8u ? (j < 4u ? i0 : i1) : (j < 12u ? i2 : i3);
        const uint32_t cls = (iw >> (8u * (j & 3u))) & 0xFFu;
        const uint32_t hi = tab[kIsingPairs + cls], lo = tab[kIsingPairs + kIsingClasses + cls];
        bool ok = hi > 65535u;  // T = 2^32
        if (!ok && lo != 0u) {
            uint32_t f[4];
            philox4x32_10(kb + j, p, rid, kTagFallback, k0, k1, f);
            ok = (f[0] & 0xFFFFu) < lo;
        }
        acc |= ok ? 1u << j : 0u;
    }
    return acc;
}

// The new own bytes nv of 4 NW sites, a whole number of Philox blocks from
// within-colour index kb on; other plane's bytes at the same place mv, at the
// side sv, above Uv and below Dv.
// About 165 VALU slots for 16 sites, 108 of them the two Philox blocks; a lookup
// and a 32-bit compare for every site took 213.
template <int NW>
__device__ __forceinline__ void ising_core(const uint32_t (&ov)[NW], const uint32_t (&mv)[NW],
                                           const uint32_t (&sv)[NW], const uint32_t (&Uv)[NW],
                                           const uint32_t (&Dv)[NW], uint32_t kb, uint32_t p,
                                           uint32_t rid, uint32_t k0, uint32_t k1,
                                           const uint32_t* tab, uint32_t (&nv)[NW]) {
    // class 9u + 3nx + ny per byte (< 18)
    uint32_t idx[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        const uint32_t nx = mv[k] + sv[k];
        idx[k] = ((ov[k] << 3) + ov[k]) + ((nx << 1) + nx) + (Uv[k] + Dv[k]);
    }
    uint32_t w[2 * NW];
#pragma unroll
    for (int b = 0; b < NW / 2; ++b)
        philox4x32_10<0x80008000u>((kb >> 3) + (uint32_t)b, p, rid, kTagMain, k0, k1, &w[4 * b]);
    const uint32_t base = (uint32_t)(uintptr_t)(lds_u32_t)tab;
    s16x2_t d[2 * NW];
    u16x2_t dmin = {0xFFFF, 0xFFFF};
#pragma unroll
    for (int i = 0; i < 2 * NW; ++i) {
        const uint32_t at =
            __builtin_amdgcn_udot4(idx[i >> 1], (i & 1) ? 0x04480000u : 0x00000448u, base, false);
        const uint32_t T = *(lds_u32_t)(uintptr_t)at;
        d[i] = __builtin_elementwise_sub_sat(__builtin_bit_cast(s16x2_t, w[i]),
                                             __builtin_bit_cast(s16x2_t, T));
        dmin = __builtin_elementwise_min(dmin, __builtin_bit_cast(u16x2_t, d[i]));
    }
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        // v_perm_b32 selectors 8 .. 11: the signs of the four 16-bit halves
        const uint32_t f = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, d[2 * k + 1]),
                                                 __builtin_bit_cast(uint32_t, d[2 * k]), 0x0B0A0908u);
        nv[k] = ov[k] ^ (f & 0x01010101u);
    }
    if (min((uint32_t)dmin.x, (uint32_t)dmin.y) == 0u) {
        uint32_t tie = 0u;
#pragma unroll
        for (int i = 0; i < 2 * NW; ++i)
            tie |= (d[i].x == 0 ? 1u << (2 * i) : 0u) | (d[i].y == 0 ? 2u << (2 * i) : 0u);
        const uint32_t acc = ising_ties(tie, tab, idx, kb, p, rid, k0, k1);
#pragma unroll
        for (int j = 0; j < 4 * NW; ++j) nv[j >> 2] ^= ((acc >> j) & 1u) << (8 * (j & 3));
    }
}

// Adds an item of a recorded sweep's colour-1 pass to byte-wise counts: up
// spins of both colours, unequal horizontal and vertical bonds (every bond has
// exactly one colour-1 end).  At most 2 NW a byte and call.
template <int NW>
__device__ __forceinline__ void ising_count(const uint32_t (&nv)[NW], const uint32_t (&mv)[NW],
                                            const uint32_t (&sv)[NW], const uint32_t (&Uv)[NW],
                                            const uint32_t (&Dv)[NW], uint32_t& up, uint32_t& dx,
                                            uint32_t& dy) {
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        up = nv[k] + mv[k] + up;
        dx = (nv[k] ^ mv[k]) + dx;
        dx = (nv[k] ^ sv[k]) + dx;
        dy = (nv[k] ^ Uv[k]) + dy;
        dy = (nv[k] ^ Dv[k]) + dy;
    }
}

__device__ __forceinline__ void arr(const uint4& v, uint32_t (&o)[4]) {
    o[0] = v.x;
    o[1] = v.y;
    o[2] = v.z;
    o[3] = v.w;
}

template <int PAR, bool REC, bool NT>
__device__ __forceinline__ void ising_compute(const ChunkIn& in, uint8_t* own, uint32_t oo,
                                              uint32_t p, uint32_t rid, uint32_t k0, uint32_t k1,
                                              const uint32_t* tab, IsingAcc& acc) {
    uint32_t ov[4], mv[4], Uv[4], Dv[4], nv[4], sv[4];
    arr(in.o, ov);
    arr(in.m, mv);
    arr(in.U, Uv);
    arr(in.D, Dv);
    side_bytes(PAR, mv, in.e, sv);
    ising_core(ov, mv, sv, Uv, Dv, oo, p, rid, k0, k1, tab, nv);
    store_own<NT>(own + oo, nv[0], nv[1], nv[2], nv[3]);
    if (REC) {
        uint32_t up = 0u, dx = 0u, dy = 0u;
        ising_count(nv, mv, sv, Uv, Dv, up, dx, dy);
        acc.M += 2 * (int)sad_u8(up, 0u) - 32;
        acc.Bx += 32 - 2 * (int)sad_u8(dx, 0u);
        acc.By += 32 - 2 * (int)sad_u8(dy, 0u);
    }
}

// ---------------------------------------------------------------- Potts
// Thresholds of a replica in LDS: the high halves by pattern (kPottsFast), then
// 9 high and 9 low halves by dn + 4 (h = 0), then, for the others, the whole
// table [tab_n hi | tab_n lo].
constexpr int kPatternWords = 256;
static_assert(kPottsTabWords == kPatternWords + 20, "table layout");

// The rule of a replica: labels of three bits and no field; no field; any.
enum { kPottsFast = 0, kPottsNoField = 1, kPottsAny = 2 };
__device__ __forceinline__ int potts_path(const RepDev& R) {
    return R.h != 0.0f ? kPottsAny : (R.q <= 8 ? kPottsFast : kPottsNoField);
}

// Lanes tid = 0 .. nthr - 1 fill l; no other lane reads before they meet.
__device__ __forceinline__ void load_potts_table(const uint32_t* tab, const RepDev& R, uint32_t* l,
                                                 int tid, int nthr) {
    const uint32_t* t = tab + R.tab_off;
    const int wq = 2 * R.q - 1;  // h = 0: the column s' = s stands for all
    if (R.h == 0.0f) {
        for (int i = tid; i < (R.q <= 8 ? kPatternWords : 0); i += nthr)
            l[i] = t[(__popc(i & 15) + 4 - __popc(i >> 4)) * wq + R.q - 1];
        for (int i = tid; i < 18; i += nthr) {
            const int k = i % 9, half = i / 9;
            l[kPatternWords + i] = t[half * R.tab_n + k * wq + R.q - 1];
        }
    } else {
        for (int i = tid; i < 2 * R.tab_n; i += nthr) l[kPottsTabWords + i] = t[i];
    }
}

struct PottsAcc {
    int Nx, Ny, S;
    int n[8];  // labels 0 .. 7 (q <= 8)
    __device__ __forceinline__ void clear() {
        Nx = Ny = S = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) n[k] = 0;
    }
};

// Byte-wise "not equal" flags (bit 7 of each byte) for labels < 128.
__device__ __forceinline__ uint32_t ne_hi(uint32_t a, uint32_t b) {
    return ((a ^ b) + 0x7F7F7F7Fu) & 0x80808080u;
}

// a where m, b elsewhere.
__device__ __forceinline__ uint32_t bfi(uint32_t m, uint32_t a, uint32_t b) {
    return __builtin_amdgcn_bitop3_b32(m, a, b, 0xCA);
}

// Word j >> 2 of NW (2 or 4), by value.
template <int NW>
__device__ __forceinline__ uint32_t word_of(const uint32_t (&v)[NW], uint32_t j) {
    const uint32_t a = v[0], b = v[1], c = v[NW - 2], d = v[NW - 1];
    return j < 8u ? (j < 4u ? a : b) : (j < 12u ? c : d);
}

// 4 NW sites, a whole number of Philox blocks from within-colour index kb on;
// neighbours as in ising_core.  About 430 VALU slots for 16 sites (kPottsFast), 220
// of them the four Philox blocks; counting neighbours flag by flag takes 520.  Passes
// over lattices in memory gain little (64 of 1024 x 1024: 29 us, 100 MB at 3.5 TB/s), but
// recorded ones do: 59 -> 35 us a pass for q = 4, the labels counted from bit planes.
template <int NW, int PATH>
__device__ __forceinline__ void potts_core(const uint32_t (&ov)[NW], const uint32_t (&mv)[NW],
                                           const uint32_t (&sv)[NW], const uint32_t (&Uv)[NW],
                                           const uint32_t (&Dv)[NW], uint32_t kb, uint32_t p,
                                           uint32_t rid, uint32_t k0, uint32_t k1,
                                           const uint32_t* tab, int q, int ntab, uint32_t lem_thr,
                                           uint32_t (&nv)[NW]) {
    constexpr int NS = 4 * NW;
    uint32_t w[NS];
#pragma unroll
    for (int b = 0; b < NW; ++b)
        philox4x32_10((kb >> 2) + (uint32_t)b, p, rid, kTagMain, k0, k1, &w[4 * b]);
    const uint32_t mq = (uint32_t)(q - 1);
    // proposals s' = s + 1 + off (mod q), off uniform in [0, q-1): off is
    // byte 2 of the 16-bit Lemire product (< 2^24), and the smallest low half
    // of the products flags a rejection anywhere
    uint32_t pr[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) pr[j] = __umul24(w[j] & 0xFFFFu, mq);  // full-rate 24-bit multiply
    // Bytewise: t = s + 1 + off <= 2q - 2 < 256; u = t + (128 - q) has bit 7
    // set iff t >= q (and stays below 256); those bytes take t - q.
    const uint32_t Cb = (uint32_t)(128 - q) * 0x01010101u;
    const uint32_t Cb1 = Cb + 0x01010101u;
    uint32_t s2v[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        const uint32_t offs = __builtin_amdgcn_perm(pr[4 * k + 1], pr[4 * k], 0x0C0C0602u) |
                              __builtin_amdgcn_perm(pr[4 * k + 3], pr[4 * k + 2], 0x06020C0Cu);
        const uint32_t u = ov[k] + offs + Cb1;
        const uint32_t G = u & 0x80808080u;
        if (PATH == kPottsFast || q <= 64) {
            // t < 128: the bytes with t >= q take the low seven bits of u
            // (u - 128 = t - q), the others u - (128 - q) = t, in one select
            s2v[k] = bfi(G - (G >> 7), u, u - Cb);
        } else {
            const uint32_t Qb = (uint32_t)q * 0x01010101u;
            s2v[k] = u - Cb - (((G << 1) - (G >> 7)) & Qb);
        }
    }
    // a rejected 16-bit Lemire draw (low half of the product below
    // 2^16 mod (q - 1)) is redrawn from the fallback stream; none are
    // rejected when q - 1 divides 2^16
    if (lem_thr != 0u) {
        uint16_t lmin = 0xFFFF;
#pragma unroll
        for (int j = 0; j < NS; ++j) lmin = min(lmin, (uint16_t)pr[j]);
        if (lmin < lem_thr) {
            uint32_t redo = 0u;
#pragma unroll
            for (int j = 0; j < NS; ++j) redo |= (pr[j] & 0xFFFFu) < lem_thr ? 1u << j : 0u;
            while (redo != 0u) {
                const uint32_t j = (uint32_t)__builtin_ctz(redo), sh = 8u * (j & 3u);
                redo &= redo - 1u;
                uint32_t f[4];
                philox4x32_10(kb + j, p, rid, kTagFallback, k0, k1, f);
                const uint32_t off = (uint32_t)(((uint64_t)f[1] * (uint64_t)mq) >> 32);
                const uint32_t t = ((word_of(ov, j) >> sh) & 0xFFu) + 1u + off;
                const uint32_t x = min(t, t - (uint32_t)q) << sh;
#pragma unroll
                for (int k = 0; k < NW; ++k)
                    s2v[k] = bfi((j >> 2) == (uint32_t)k ? 0xFFu << sh : 0u, x, s2v[k]);
            }
        }
    }
    // The class of a site by dn + 4 = #ne(s) + #eq(s'), per byte of cls.
    uint32_t cls[NW];
    if (PATH == kPottsFast) {
        // s and s' side by side in the nibbles of a byte, compared with a
        // neighbour at once: bit 3 of each nibble of (x ^ c) + 7 is set iff they
        // differ.  The four neighbours' flags gather in a nibble each: the
        // pattern of a site, whose threshold the table holds.
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const uint32_t x = ov[k] | (s2v[k] << 4);
            const uint32_t t0 = (x ^ (mv[k] | (mv[k] << 4))) + 0x77777777u;
            const uint32_t t1 = (x ^ (sv[k] | (sv[k] << 4))) + 0x77777777u;
            const uint32_t t2 = (x ^ (Uv[k] | (Uv[k] << 4))) + 0x77777777u;
            const uint32_t t3 = (x ^ (Dv[k] | (Dv[k] << 4))) + 0x77777777u;
            const uint32_t a = bfi(0x88888888u, t0, t1 >> 1), b = bfi(0x88888888u, t2, t3 >> 1);
            cls[k] = bfi(0xCCCCCCCCu, a, b >> 2);
        }
    } else if (q <= 16) {
        // Labels below 2^b (b <= 4): ((a ^ c) + (2^b - 1)) has bit b set iff
        // a != c; the eight flags (unequal to s, equal to s') sum to
        // (4 + dn) 2^b < 256 in each byte, so no per-flag shift is needed.
        const int b = q <= 2 ? 1 : 32 - __clz(q - 1);
        const uint32_t F = 0x01010101u << b, A = F - 0x01010101u;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const uint32_t neo = (((ov[k] ^ mv[k]) + A) & F) + (((ov[k] ^ sv[k]) + A) & F) +
                                 (((ov[k] ^ Uv[k]) + A) & F) + (((ov[k] ^ Dv[k]) + A) & F);
            const uint32_t eqn = (~((s2v[k] ^ mv[k]) + A) & F) + (~((s2v[k] ^ sv[k]) + A) & F) +
                                 (~((s2v[k] ^ Uv[k]) + A) & F) + (~((s2v[k] ^ Dv[k]) + A) & F);
            cls[k] = (neo + eqn) >> b;
        }
    } else {
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const uint32_t neo = (ne_hi(ov[k], mv[k]) >> 7) + (ne_hi(ov[k], sv[k]) >> 7) +
                                 (ne_hi(ov[k], Uv[k]) >> 7) + (ne_hi(ov[k], Dv[k]) >> 7);
            const uint32_t nen = (ne_hi(s2v[k], mv[k]) >> 7) + (ne_hi(s2v[k], sv[k]) >> 7) +
                                 (ne_hi(s2v[k], Uv[k]) >> 7) + (ne_hi(s2v[k], Dv[k]) >> 7);
            cls[k] = neo + 0x04040404u - nen;
        }
    }
    // Threshold of pattern or dn + 4, or (with a field) of (dn + 4)(2q - 1) +
    // (s' - s + q - 1).  d = r - T_hi unsigned: bit 31 set iff the prefix
    // accepts, 0 iff it ties.
    const uint32_t wq = (uint32_t)(2 * q - 1);
    const uint32_t* t9 = tab + kPatternWords;
    const uint32_t* thr = tab + kPottsTabWords;
    const uint32_t base = (uint32_t)(uintptr_t)(lds_u32_t)(PATH == kPottsFast ? tab : t9);
    uint32_t d[NS];
    uint32_t dmin = 0xFFFFFFFFu;
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        const int sh = 8 * (j & 3);
        uint32_t th;
        if (PATH != kPottsAny) {
            const uint32_t at = __builtin_amdgcn_udot4(cls[j >> 2], 4u << sh, base, false);
            th = *(lds_u32_t)(uintptr_t)at;
        } else {
            const uint32_t s = (ov[j >> 2] >> sh) & 0xFFu;
            const uint32_t s2 = (s2v[j >> 2] >> sh) & 0xFFu;
            th = thr[__umul24((cls[j >> 2] >> sh) & 0xFFu, wq) + s2 + (uint32_t)(q - 1) - s];
        }
        d[j] = (w[j] >> 16) - th;
        dmin = min(dmin, d[j]);
    }
    uint32_t acc_sel[NW];  // 0xFF in bytes that accept
#pragma unroll
    for (int k = 0; k < NW; ++k)
        acc_sel[k] = sign_bytes(d[4 * k], d[4 * k + 1], d[4 * k + 2], d[4 * k + 3]);
    if (dmin == 0u) {
        // a prefix equals the threshold's high half: the low halves decide
        uint32_t tie = 0u;
#pragma unroll
        for (int j = 0; j < NS; ++j) tie |= d[j] == 0u ? 1u << j : 0u;
        while (tie != 0u) {
            const uint32_t j = (uint32_t)__builtin_ctz(tie), sh = 8u * (j & 3u);
            tie &= tie - 1u;
            const uint32_t c = (word_of(cls, j) >> sh) & 0xFFu;
            uint32_t lo;
            if (PATH == kPottsFast) {
                lo = t9[9u + __popc(c & 15u) + 4u - __popc(c >> 4)];
            } else if (PATH == kPottsNoField) {
                lo = t9[9u + c];
            } else {
                const uint32_t s = (word_of(ov, j) >> sh) & 0xFFu;
                const uint32_t s2 = (word_of(s2v, j) >> sh) & 0xFFu;
                lo = thr[(uint32_t)ntab + __umul24(c, wq) + s2 + (uint32_t)(q - 1) - s];
            }
            if (lo == 0u) continue;
            uint32_t f[4];
            philox4x32_10(kb + j, p, rid, kTagFallback, k0, k1, f);
            if ((f[0] & 0xFFFFu) < lo) {
#pragma unroll
                for (int k = 0; k < NW; ++k)
                    acc_sel[k] |= (j >> 2) == (uint32_t)k ? 0xFFu << sh : 0u;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < NW; ++k) nv[k] = bfi(acc_sel[k], s2v[k], ov[k]);
}

// Labels 0 .. 7 of two planes' words counted from bit planes: the labels of 8 NW
// sites as nibbles, one word a bit, and a population count for each label.
template <int NW>
__device__ __forceinline__ void count_labels8(const uint32_t (&a)[NW], const uint32_t (&b)[NW],
                                              int (&n)[8]) {
    uint32_t B[3] = {0u, 0u, 0u};
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        const uint32_t x = a[k] | (b[k] << 4);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const uint32_t m = 0x11111111u << k;
            B[i] = bfi(m, k >= i ? x << (k - i) : x >> (i - k), B[i]);
        }
    }
    constexpr uint32_t all = NW == 4 ? ~0u : 0x33333333u;
#pragma unroll
    for (int l = 0; l < 8; ++l)
        n[l] += __popc(((l & 1) ? B[0] : ~B[0]) & ((l & 2) ? B[1] : ~B[1]) &
                       ((l & 4) ? B[2] : (~B[2] & all)));
}

// Adds an item of a recorded sweep's colour-1 pass (every bond has one colour-1
// end): equal bonds, label sum and the labels of both colours, those of q > 8 by
// atomics in lhist.
template <int NW>
__device__ __forceinline__ void potts_count(const uint32_t (&nv)[NW], const uint32_t (&mv)[NW],
                                            const uint32_t (&sv)[NW], const uint32_t (&Uv)[NW],
                                            const uint32_t (&Dv)[NW], int q, PottsAcc& acc,
                                            int* lhist) {
    uint32_t nex = 0u, ney = 0u, ssum = 0u;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        nex = sad_u8((ne_hi(nv[k], mv[k]) >> 7) + (ne_hi(nv[k], sv[k]) >> 7), nex);
        ney = sad_u8((ne_hi(nv[k], Uv[k]) >> 7) + (ne_hi(nv[k], Dv[k]) >> 7), ney);
        ssum = sad_u8(nv[k], ssum);
        ssum = sad_u8(mv[k], ssum);
    }
    acc.Nx += 8 * NW - (int)nex;
    acc.Ny += 8 * NW - (int)ney;
    acc.S += (int)ssum;
    if (q <= 8) {
        count_labels8(nv, mv, acc.n);
    } else {
#pragma unroll
        for (int j = 0; j < 4 * NW; ++j) {
            atomicAdd(&lhist[(nv[j >> 2] >> (8 * (j & 3))) & 0xFFu], 1);
            atomicAdd(&lhist[(mv[j >> 2] >> (8 * (j & 3))) & 0xFFu], 1);
        }
    }
}

// Sum over the 16 lanes of a row (the n = 4 or 8 lanes of a group).
__device__ __forceinline__ int row_sum(int v, int n) {
    // quad_perm 1 0 3 2, quad_perm 2 3 0 1, row_half_mirror, row_mirror
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true);
    if (n > 4) v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true);
    if (n > 8) v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, true);
    return v;
}

// Adds acc's labels (q <= 8) to lhist and (SUM) its sums to sum[3];
// groups of n lanes (at least 16: any).  A group's lanes add one count each.
template <bool SUM>
__device__ __forceinline__ void add_counts(const PottsAcc& acc, int q, int n, int* lhist, int* sum) {
    const int m = min(n, 16), lane = (int)threadIdx.x & (m - 1);
    int v[11];
#pragma unroll
    for (int l = 0; l < 8; ++l) v[l] = q <= 8 ? row_sum(acc.n[l], n) : 0;
    v[8] = row_sum(acc.Nx, n);
    v[9] = row_sum(acc.Ny, n);
    v[10] = row_sum(acc.S, n);
    for (int k0 = 0; k0 < 11; k0 += m) {  // once where a group has 16 lanes
        const int k = k0 + lane;
        int x = v[0];
#pragma unroll
        for (int l = 1; l < 11; ++l) x = k == l ? v[l] : x;
        if (k < 8) {
            if (q <= 8) atomicAdd(&lhist[k], x);
        } else if (k < 11 && SUM) {
            atomicAdd(&sum[k - 8], x);
        }
    }
}

// 16-site Potts chunk of a plane in global memory.
// Byte offsets within a plane: oo of the chunk (own row and the other
// plane's same row), uo / dof of the rows above / below, eo of the halo dword.
template <int PAR, bool REC, int PATH, bool NT>
__device__ __forceinline__ void potts_chunk(uint8_t* own, const uint8_t* oth, uint32_t oo,
                                            uint32_t uo, uint32_t dof, uint32_t eo, uint32_t p,
                                            uint32_t rid, uint32_t k0, uint32_t k1,
                                            const uint32_t* tab, int q, int ntab, uint32_t lem_thr,
                                            PottsAcc& acc, int* lhist) {
    const ChunkIn in = chunk_load<NT>(own, oth, oo, uo, dof, eo);
    uint32_t ov[4], mv[4], Uv[4], Dv[4], nv[4], sv[4];
    arr(in.o, ov);
    arr(in.m, mv);
    arr(in.U, Uv);
    arr(in.D, Dv);
    side_bytes(PAR, mv, in.e, sv);
    potts_core<4, PATH>(ov, mv, sv, Uv, Dv, oo, p, rid, k0, k1, tab, q, ntab, lem_thr, nv);
    store_own<NT>(own + oo, nv[0], nv[1], nv[2], nv[3]);
    if (REC) potts_count(nv, mv, sv, Uv, Dv, q, acc, lhist);
}

// ------------------------------------------------- tile-level iteration
// Rows [y0, y0+rows) of plane c (y0, rows even), split over threads
// tid = 0..nthr-1 (a whole workgroup, or the share of one replica when a
// workgroup holds several).  Rows are visited by parity so that PAR is
// uniform across a wave.
template <bool REC, int PATH, bool NT>
__device__ __forceinline__ void run_tile_potts(uint8_t* planes, int W, int Ly, int y0, int rows,
                                               int c, uint32_t p, uint32_t rid, uint32_t k0,
                                               uint32_t k1, const uint32_t* tab, int q, int ntab,
                                               uint32_t lem_thr, PottsAcc& pa, int* lhist,
                                               int tid, int nthr) {
    uint8_t* own = planes + (size_t)c * Ly * W;
    const uint8_t* oth = planes + (size_t)(1 - c) * Ly * W;
    const int cpr = W >> 4;
    // item it = r * cpr + jc (row pair r, chunk column jc), advanced by nthr
    // without a division per item
    const int dr = nthr / cpr, dj = nthr - dr * cpr;
    const int r0 = tid / cpr, jc0 = tid - r0 * cpr;
    const uint32_t Wb = (uint32_t)W, W2 = 2u * Wb;
    const uint32_t last = (uint32_t)(Ly - 1) * Wb;
    // 32-bit plane offsets advanced per item: row offset ro by dr row pairs
    // (one more when the chunk column wraps), column j0 by dj chunks; the
    // row pairs of the tile end where ro reaches row y0 + rows
    const uint32_t dro = (uint32_t)dr * W2, dj0 = (uint32_t)dj << 4;
#pragma unroll
    for (int par = 0; par < 2; ++par) {
        const int yf = y0 + ((par ^ c) & 1);
        const uint32_t ro_end = (uint32_t)(yf + rows) * Wb;
        uint32_t ro = (uint32_t)(yf + 2 * r0) * Wb, j0 = (uint32_t)jc0 << 4;
        for (; ro < ro_end;) {
            if (par == 0) {
                const ChunkOff<0> f(ro, j0, Wb, last);
                potts_chunk<0, REC, PATH, NT>(own, oth, f.oo, f.uo, f.dof, f.eo, p, rid, k0, k1,
                                              tab, q, ntab, lem_thr, pa, lhist);
            } else {
                const ChunkOff<1> f(ro, j0, Wb, last);
                potts_chunk<1, REC, PATH, NT>(own, oth, f.oo, f.uo, f.dof, f.eo, p, rid, k0, k1,
                                              tab, q, ntab, lem_thr, pa, lhist);
            }
            ro += dro;
            j0 += dj0;
            if (j0 >= Wb) {
                j0 -= Wb;
                ro += W2;
            }
        }
    }
}

// Ising rows [y0, y0+rows) of plane c.  Each lane takes one chunk of each row
// parity per iteration and issues both chunks' loads before computing (latency
// hiding for the HBM stream).
template <bool REC, bool NT>
__device__ __forceinline__ void run_tile_ising(uint8_t* planes, int W, int Ly, int y0, int rows,
                                               int c, uint32_t p, uint32_t rid, uint32_t k0,
                                               uint32_t k1, const uint32_t* thr, IsingAcc& ia,
                                               int tid, int nthr) {
    uint8_t* own = planes + (size_t)c * Ly * W;
    const uint8_t* oth = planes + (size_t)(1 - c) * Ly * W;
    const int cpr = W >> 4;
    const int ya = y0 + (c & 1);        // rows with (y + c) & 1 == 0
    const int yb = y0 + ((c & 1) ^ 1);  // rows with (y + c) & 1 == 1
    // item it = r * cpr + jc (row pair r, chunk column jc), advanced by nthr
    // without a division per item: the 32-bit row offset by dr row pairs (one
    // more when the column wraps), the column by dj chunks; the row pairs of
    // the tile end where the row offset reaches row y0 + rows
    const int dr = nthr / cpr, dj = nthr - dr * cpr;
    const int r0 = tid / cpr, jc0 = tid - r0 * cpr;
    const uint32_t Wb = (uint32_t)W, W2 = 2u * Wb;
    const uint32_t last = (uint32_t)(Ly - 1) * Wb;
    const uint32_t dro = (uint32_t)dr * W2, dj0 = (uint32_t)dj << 4;
    // ra: row of parity 0, ra + db: the row of parity 1 in the same pair
    const int db = yb - ya;  // +1 or -1
    const uint32_t ra_end = (uint32_t)(ya + rows) * Wb;
    uint32_t ra = (uint32_t)(ya + 2 * r0) * Wb, j0 = (uint32_t)jc0 << 4;
    for (; ra < ra_end;) {
        const uint32_t rb = ra + (uint32_t)db * Wb;
        const ChunkOff<0> fa(ra, j0, Wb, last);
        const ChunkOff<1> fb(rb, j0, Wb, last);
        const ChunkIn A = chunk_load<NT>(own, oth, fa.oo, fa.uo, fa.dof, fa.eo);
        const ChunkIn B = chunk_load<NT>(own, oth, fb.oo, fb.uo, fb.dof, fb.eo);
        ising_compute<0, REC, NT>(A, own, fa.oo, p, rid, k0, k1, thr, ia);
        ising_compute<1, REC, NT>(B, own, fb.oo, p, rid, k0, k1, thr, ia);
        ra += dro;
        j0 += dj0;
        if (j0 >= Wb) {
            j0 -= Wb;
            ra += W2;
        }
    }
}

__device__ __forceinline__ void load_table(const uint32_t* tab, const RepDev& R, uint32_t* lthr,
                                           int tid, int nthr) {
    const int n2 = 2 * R.tab_n;
    for (int i = tid; i < n2; i += nthr) lthr[i] = tab[R.tab_off + i];
}

__device__ __forceinline__ uint32_t lemire_threshold(int q) {
    return 65536u % (uint32_t)(q - 1);
}

// Potts tile with the rule chosen per replica.
template <bool REC, bool NT>
__device__ __forceinline__ void potts_tile(const RepDev& R, uint8_t* planes, int y0, int rows,
                                           int c, uint32_t p, uint32_t k0, uint32_t k1,
                                           const uint32_t* tab, PottsAcc& pa, int* lhist, int tid,
                                           int nthr) {
    const uint32_t lt = lemire_threshold(R.q);
    const int path = potts_path(R);
    if (path == kPottsFast)
        run_tile_potts<REC, kPottsFast, NT>(planes, R.W, R.Ly, y0, rows, c, p, R.rid, k0, k1, tab,
                                            R.q, R.tab_n, lt, pa, lhist, tid, nthr);
    else if (path == kPottsNoField)
        run_tile_potts<REC, kPottsNoField, NT>(planes, R.W, R.Ly, y0, rows, c, p, R.rid, k0, k1,
                                               tab, R.q, R.tab_n, lt, pa, lhist, tid, nthr);
    else
        run_tile_potts<REC, kPottsAny, NT>(planes, R.W, R.Ly, y0, rows, c, p, R.rid, k0, k1, tab,
                                           R.q, R.tab_n, lt, pa, lhist, tid, nthr);
}

// XCD-aware block order: consecutive logical units land on one XCD (blocks
// are dispatched round-robin over the 8 XCDs), so neighbouring row tiles of a
// replica share that XCD's L2.
__device__ __forceinline__ int logical_block(int n) {
    const int b = blockIdx.x;
    if ((n & 7) != 0) return b;
    return (b & 7) * (n >> 3) + (b >> 3);
}


}  // namespace

// ---------------------------------------------------------------- kernels
// One colour pass over the row tiles [tile0, tile0 + n) of one model.  The
// two models have separate kernels so that each gets its own register
// budget (Ising needs about half of Potts's, hence twice the waves per SIMD).
template <int MODEL, bool NT>
__device__ __forceinline__ void stream_pass_body(const SweepArgs& a, int tile0, int n, int c,
                                                 int sweep_off, int rec_row, uint32_t* lthr,
                                                 int* lhist, int* lred) {
    const TileDev T = a.tiles[tile0 + logical_block(n)];
    const RepDev R = a.reps[T.rep];
    if (MODEL == kModelPotts) {
        load_potts_table(a.tab, R, lthr, threadIdx.x, blockDim.x);
    } else {
        load_ising_table(a.tab, R, lthr, threadIdx.x, blockDim.x);
    }
    const bool rec = (rec_row >= 0) && (c == 1);
    if (MODEL == kModelPotts && rec)
        for (int i = threadIdx.x; i < max(R.q, 8); i += blockDim.x) lhist[i] = 0;
    __syncthreads();
    const uint64_t t = *a.t_base + (uint64_t)sweep_off;
    const uint32_t p = (uint32_t)(2 * t + (uint64_t)c);
    uint8_t* planes = a.lat + R.lat_off;
    IsingAcc ia{0, 0, 0};
    PottsAcc pa;
    pa.clear();
    if (MODEL == kModelIsing) {
        if (rec)
            run_tile_ising<true, NT>(planes, R.W, R.Ly, T.y0, T.rows, c, p, R.rid, a.key0, a.key1,
                                 lthr, ia, threadIdx.x, blockDim.x);
        else
            run_tile_ising<false, NT>(planes, R.W, R.Ly, T.y0, T.rows, c, p, R.rid, a.key0, a.key1,
                                  lthr, ia, threadIdx.x, blockDim.x);
    } else {
        if (rec)
            potts_tile<true, NT>(R, planes, T.y0, T.rows, c, p, a.key0, a.key1, lthr, pa, lhist,
                                 threadIdx.x, blockDim.x);
        else
            potts_tile<false, NT>(R, planes, T.y0, T.rows, c, p, a.key0, a.key1, lthr, pa, lhist,
                                  threadIdx.x, blockDim.x);
    }
    if (rec) {
        int v[3];
        if (MODEL == kModelIsing) {
            v[0] = ia.M; v[1] = ia.Bx; v[2] = ia.By;
        } else {
            v[0] = pa.Nx; v[1] = pa.Ny; v[2] = pa.S;
        }
        if (MODEL == kModelPotts && R.q <= 8) add_counts<false>(pa, R.q, 64, lhist, nullptr);
        block_sum<3>(v, lred);
        int32_t* row = a.stats + ((size_t)rec_row * a.R + T.rep) * a.width;
        if (threadIdx.x == 0) {
            atomicAdd(&row[0], v[0]);
            atomicAdd(&row[1], v[1]);
            atomicAdd(&row[2], v[2]);
        }
        if (MODEL == kModelPotts) {
            __syncthreads();
            for (int i = threadIdx.x; i < R.q; i += blockDim.x)
                if (lhist[i]) atomicAdd(&a.hist[R.hist_off + i], lhist[i]);
        }
    }
}

// Occupancy targets: the Ising pass is memory-streaming and wants many
// waves in flight; the Potts pass is VALU-heavy and keeps more registers.
template <bool NT>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(6, 8)))
k_stream_pass_ising(SweepArgs a, int tile0, int n, int c, int sweep_off, int rec_row) {
    __shared__ uint32_t tab[kIsingTabWords];  // thresholds of this tile's replica
    __shared__ int lred[64];
    stream_pass_body<kModelIsing, NT>(a, tile0, n, c, sweep_off, rec_row, tab, nullptr, lred);
}

template <bool NT>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(3, 8)))
k_stream_pass_potts(SweepArgs a, int tile0, int n, int c, int sweep_off, int rec_row) {
    extern __shared__ uint32_t lthr[];  // kPottsTabWords, with fields the whole table too
    __shared__ int lhist[kMaxPottsQ];
    __shared__ int lred[64];
    stream_pass_body<kModelPotts, NT>(a, tile0, n, c, sweep_off, rec_row, lthr, lhist, lred);
}

// ------------------------------------------------- persistent streamed passes
// One launch runs every colour pass of a chunk of unrecorded sweeps over the
// streamed replicas of one model (the batched scheduler without a launch per
// pass).  Workgroup g owns its items for the whole launch: whole replicas,
// which no other workgroup touches, so the workgroup's barrier between
// passes orders their passes, or one row slab of a replica cut into slabs
// owned by different workgroups.  A slab's pass j (counted from 0 within the
// launch) reads the other plane's rows just above and below it, which the
// neighbouring slabs write in their pass j - 1, and writes rows that they
// read in their pass j - 1; so it starts once both neighbours have published
// pass j - 1 (flag >= j), and a slab never runs more than one pass ahead of
// its neighbours.  Publishing: every lane waits for its stores, the
// workgroup meets at a barrier, lane 0 stores flag = j + 1 with agent-scope
// release (write-back of the XCD's L2).  Waiting: lane 0 polls the
// neighbours' flags, then takes an agent-scope acquire (invalidation of its
// L1 and L2) before the barrier that lets the other lanes read.  All slab
// workgroups must be resident at once: the host keeps their number within
// the occupancy of the whole chip and numbers them first, so that in-order
// dispatch places them before any whole-replica workgroup.  A wait that
// exceeds its bound (about two seconds) raises *abort, and every waiting
// workgroup then leaves: a launch always ends.
constexpr uint32_t kPersistSpinCap = 1u << 25;  // polls of ~128 cycles each

// every store of this lane has completed (vmcnt 0; exp and lgkm counts
// left at their maxima)
__device__ __forceinline__ void wait_stores() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Agent-scope release of a pass flag: the fence writes the L2 back (the
// workgroup's rows reach memory for the other XCDs), the explicit vmcnt(0)
// waits for that write-back to finish, then the flag is stored.  (The
// release store alone compiles to the write-back directly followed by the
// flag store, with no wait between them, when the workgroup's stores were
// already waited for, so the flag could be seen before the rows.)
__device__ __forceinline__ void persist_publish(uint32_t* flag, uint32_t v) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    wait_stores();
    __hip_atomic_store(flag, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ int persist_wait(uint32_t* flags, int up, int down, uint32_t need, uint32_t* abort_flag) {
    for (uint32_t spin = 0;; ++spin) {
        const uint32_t u = __hip_atomic_load(&flags[up], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t d = __hip_atomic_load(&flags[down], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (u >= need && d >= need) break;
        if (__hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) return 0;
        if (spin >= kPersistSpinCap) {
            __hip_atomic_store(abort_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return 0;
        }
        __builtin_amdgcn_s_sleep(2);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return 1;
}

template <int MODEL, bool NT>
__device__ __forceinline__ void persist_body(const SweepArgs& a, const PersistItem* items,
                                             const int32_t* item_off, uint32_t* flags,
                                             uint32_t* abort_flag, int slot_words, uint32_t* lds,
                                             int* go) {
    const int i0 = item_off[blockIdx.x], i1 = item_off[blockIdx.x + 1];
    // threshold tables of the items' replicas
    for (int k = i0; k < i1; ++k) {
        const RepDev R = a.reps[items[k].rep];
        uint32_t* t = lds + (k - i0) * slot_words;
        if (MODEL == kModelPotts) {
            load_potts_table(a.tab, R, t, threadIdx.x, blockDim.x);
        } else {
            load_ising_table(a.tab, R, t, threadIdx.x, blockDim.x);
        }
    }
    __syncthreads();
    const uint64_t t0 = *a.t_base + (uint64_t)a.sweep_off;
    for (int sw = 0; sw < a.n_sweeps; ++sw) {
        for (int c = 0; c < 2; ++c) {
            const uint32_t j = (uint32_t)(2 * sw + c);
            const uint32_t p = (uint32_t)(2 * (t0 + (uint64_t)sw) + (uint64_t)c);
            for (int k = i0; k < i1; ++k) {
                const PersistItem it = items[k];
                if (it.slab >= 0 && j > 0) {
                    if (threadIdx.x == 0) *go = persist_wait(flags, it.up, it.down, j, abort_flag);
                    __syncthreads();
                    if (!*go) return;  // uniform: the whole workgroup leaves
                }
                const RepDev R = a.reps[it.rep];
                uint32_t* tab = lds + (k - i0) * slot_words;
                uint8_t* planes = a.lat + R.lat_off;
                if (MODEL == kModelIsing) {
                    IsingAcc ia{0, 0, 0};
                    run_tile_ising<false, NT>(planes, R.W, R.Ly, it.y0, it.rows, c, p, R.rid,
                                                    a.key0, a.key1, tab, ia, threadIdx.x,
                                                    blockDim.x);
                } else {
                    PottsAcc pa;
                    pa.clear();
                    potts_tile<false, NT>(R, planes, it.y0, it.rows, c, p, a.key0, a.key1, tab, pa,
                                          nullptr, threadIdx.x, blockDim.x);
                }
                if (it.slab >= 0) {
                    wait_stores();
                    __syncthreads();
                    if (threadIdx.x == 0) persist_publish(&flags[it.slab], j + 1u);
                }
            }
            __syncthreads();  // the workgroup's pass boundary
        }
    }
}

template <bool NT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6, 8)))
k_persist_ising(SweepArgs a, const PersistItem* items, const int32_t* item_off, uint32_t* flags,
                uint32_t* abort_flag, int slot_words) {
    extern __shared__ uint32_t ptab[];
    __shared__ int go;
    persist_body<kModelIsing, NT>(a, items, item_off, flags, abort_flag, slot_words, ptab, &go);
}

template <bool NT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 8)))
k_persist_potts(SweepArgs a, const PersistItem* items, const int32_t* item_off, uint32_t* flags,
                uint32_t* abort_flag, int slot_words) {
    extern __shared__ uint32_t ptab[];
    __shared__ int go;
    persist_body<kModelPotts, NT>(a, items, item_off, flags, abort_flag, slot_words, ptab, &go);
}

// nmax of each Potts replica from its histogram; clears the histogram.
__global__ void k_potts_hist_finalize(SweepArgs a, const int32_t* list, int n, int rec_row) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int r = list[i];
    const RepDev R = a.reps[r];
    int mx = 0;
    for (int k = 0; k < R.q; ++k) {
        const int v = a.hist[R.hist_off + k];
        mx = v > mx ? v : mx;
        a.hist[R.hist_off + k] = 0;
    }
    a.stats[((size_t)rec_row * a.R + r) * a.width + 3] = mx;
}

// ------------------------------------------------------ generic (any L)
namespace {

__device__ __forceinline__ int wrapi(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// One site of colour c, within-colour index k, in planes (LDS or global).
__device__ __forceinline__ void generic_site(int model, uint8_t* planes, int W, int Ly, int c,
                                             int k, uint32_t p, uint32_t rid, uint32_t k0,
                                             uint32_t k1, const uint32_t* thr, int q, int ntab) {
    const int y = k / W;
    const int j = k - y * W;
    const int off = (y + c) & 1;
    uint8_t* own = planes + (size_t)c * Ly * W;
    const uint8_t* oth = planes + (size_t)(1 - c) * Ly * W;
    const int ym = wrapi(y - 1, Ly), yp = wrapi(y + 1, Ly);
    const int js = wrapi(off ? j + 1 : j - 1, W);
    const uint32_t s = own[(size_t)y * W + j];
    const uint32_t a0 = oth[(size_t)y * W + j], a1 = oth[(size_t)y * W + js];
    const uint32_t b0 = oth[(size_t)ym * W + j], b1 = oth[(size_t)yp * W + j];
    uint32_t w[4];
    if (model == kModelIsing) {
        philox4x32_10((uint32_t)k >> 3, p, rid, kTagMain, k0, k1, w);
        const uint32_t h = (uint32_t)k & 7u;
        const uint32_t r = (w[h >> 1] >> (16 * (h & 1))) & 0xFFFFu;
        const uint32_t cls = 9u * s + 3u * (a0 + a1) + (b0 + b1);
        const uint32_t hi = thr[cls];
        bool acc = r < hi;
        if (r == hi && thr[kIsingClasses + cls] != 0u) {
            uint32_t f[4];
            philox4x32_10((uint32_t)k, p, rid, kTagFallback, k0, k1, f);
            acc = (f[0] & 0xFFFFu) < thr[kIsingClasses + cls];
        }
        if (acc) own[(size_t)y * W + j] = (uint8_t)(s ^ 1u);
    } else {
        philox4x32_10((uint32_t)k >> 2, p, rid, kTagMain, k0, k1, w);
        const uint32_t word = w[k & 3];
        const uint32_t mq = (uint32_t)(q - 1);
        const uint32_t prod = (word & 0xFFFFu) * mq;
        uint32_t off2 = prod >> 16;
        uint32_t f[4];
        bool have_f = false;
        if ((prod & 0xFFFFu) < 65536u % mq) {
            philox4x32_10((uint32_t)k, p, rid, kTagFallback, k0, k1, f);
            have_f = true;
            off2 = (uint32_t)(((uint64_t)f[1] * (uint64_t)mq) >> 32);
        }
        uint32_t s2 = s + 1u + off2;
        s2 = s2 >= (uint32_t)q ? s2 - (uint32_t)q : s2;
        const int dn = (int)(a0 == s2) + (int)(a1 == s2) + (int)(b0 == s2) + (int)(b1 == s2) -
                       (int)(a0 == s) - (int)(a1 == s) - (int)(b0 == s) - (int)(b1 == s);
        const uint32_t cls = (uint32_t)(dn + 4) * (uint32_t)(2 * q - 1) + s2 + (uint32_t)(q - 1) - s;
        const uint32_t hi = thr[cls];
        const uint32_t r = word >> 16;
        bool acc = r < hi;
        if (r == hi && thr[ntab + cls] != 0u) {
            if (!have_f) philox4x32_10((uint32_t)k, p, rid, kTagFallback, k0, k1, f);
            acc = (f[0] & 0xFFFFu) < thr[ntab + cls];
        }
        if (acc) own[(size_t)y * W + j] = (uint8_t)s2;
    }
}

__device__ __forceinline__ uint32_t site_at(const uint8_t* planes, int W, int Ly, int y, int x) {
    return planes[(size_t)((x + y) & 1) * Ly * W + (size_t)y * W + (x >> 1)];
}

// Integer statistics of a whole lattice (Ising: M, Bx, By; Potts: Nx, Ny, S
// and the label histogram into hist).  Thread-strided over natural sites.
__device__ __forceinline__ void lattice_stats(int model, const uint8_t* planes, int Lx, int Ly,
                                              int W, int n0, int n1, int (&v)[3], int* hist) {
    for (int n = n0 + (int)threadIdx.x; n < n1; n += blockDim.x) {
        const int y = n / Lx, x = n - y * Lx;
        const int s = (int)site_at(planes, W, Ly, y, x);
        const int r = (int)site_at(planes, W, Ly, y, x + 1 == Lx ? 0 : x + 1);
        const int d = (int)site_at(planes, W, Ly, y + 1 == Ly ? 0 : y + 1, x);
        if (model == kModelIsing) {
            const int ss = 2 * s - 1;
            v[0] += ss;
            v[1] += ss * (2 * r - 1);
            v[2] += ss * (2 * d - 1);
        } else {
            v[0] += (s == r);
            v[1] += (s == d);
            v[2] += s;
            atomicAdd(&hist[s], 1);
        }
    }
}

}  // namespace

// Resident kernel: a workgroup owns a.rpb replicas of one shape for the
// whole call, each with its thresholds and both planes in LDS, and
// blockDim/rpb threads; colour passes are separated by workgroup barriers.
// Site by site for any model and width: lattices narrower than 16 (plane rows
// below 8 bytes); all others have the kernels of items below.
__global__ void __launch_bounds__(512) k_resident_generic(SweepArgs a) {
    // dynamic LDS: rpb slots of [thresholds (tab_lds_bytes) | plane 0 | plane 1]
    extern __shared__ __align__(16) uint8_t dyn[];
    __shared__ int lhist[kMaxPottsQ];
    __shared__ int lred[64];
    const int P = a.rpb;
    const int nt = blockDim.x / P;
    const int g = threadIdx.x / nt, lt = threadIdx.x - g * nt;
    const int first = blockIdx.x * P;
    const bool active = g < P && first + g < a.n_list;
    const int rep = a.rep_list[active ? first + g : first];
    const RepDev R = a.reps[rep];
    uint8_t* slot = dyn + (size_t)(active ? g : 0) * a.res_slot_bytes;
    uint32_t* lthr = reinterpret_cast<uint32_t*>(slot);
    uint8_t* lds = slot + a.tab_lds_bytes;
    const int plane = R.Ly * R.W;
    const int bytes = 2 * plane;
    uint8_t* gmem = a.lat + R.lat_off;
    if (active) {
        if ((bytes & 15) == 0) {
            for (int i = lt; i < (bytes >> 4); i += nt)
                reinterpret_cast<uint4*>(lds)[i] = reinterpret_cast<const uint4*>(gmem)[i];
        } else {
            for (int i = lt; i < bytes; i += nt) lds[i] = gmem[i];
        }
        load_table(a.tab, R, lthr, lt, nt);
    }
    __syncthreads();
    const uint64_t t0 = *a.t_base;
    for (int i = 0; i < a.n_sweeps; ++i) {
        const int sw = a.sweep_off + i;  // sweep index within the call
        const uint64_t t = t0 + (uint64_t)sw;
        const bool rec = a.record_every > 0 && ((sw + 1) % a.record_every) == 0;
        for (int c = 0; c < 2; ++c) {
            const uint32_t p = (uint32_t)(2 * t + (uint64_t)c);
            if (active) {
                for (int k = lt; k < plane; k += nt)
                    generic_site(R.model, lds, R.W, R.Ly, c, k, p, R.rid, a.key0, a.key1, lthr,
                                 R.q, R.tab_n);
            }
            __syncthreads();
        }
        if (rec) {
            // statistics of each replica of the workgroup, all threads per replica
            for (int gg = 0; gg < P && first + gg < a.n_list; ++gg) {
                const int rg = a.rep_list[first + gg];
                const RepDev Q = a.reps[rg];
                const uint8_t* lq = dyn + (size_t)gg * a.res_slot_bytes + a.tab_lds_bytes;
                if (Q.model == kModelPotts) {
                    for (int k = threadIdx.x; k < Q.q; k += blockDim.x) lhist[k] = 0;
                    __syncthreads();
                }
                int v[3] = {0, 0, 0};
                lattice_stats(Q.model, lq, Q.Lx, Q.Ly, Q.W, 0, Q.Lx * Q.Ly, v, lhist);
                block_sum<3>(v, lred);
                int32_t* row =
                    a.stats + ((size_t)((sw + 1) / a.record_every - 1) * a.R + rg) * a.width;
                if (threadIdx.x == 0) {
                    row[0] = v[0];
                    row[1] = v[1];
                    row[2] = v[2];
                    int mx = 0;
                    if (Q.model == kModelPotts)
                        for (int k = 0; k < Q.q; ++k) mx = lhist[k] > mx ? lhist[k] : mx;
                    row[3] = mx;
                    for (int k = 4; k < a.width; ++k) row[k] = 0;
                }
                __syncthreads();
            }
        }
    }
    if (active) {
        if ((bytes & 15) == 0) {
            for (int i = lt; i < (bytes >> 4); i += nt)
                reinterpret_cast<uint4*>(gmem)[i] = reinterpret_cast<const uint4*>(lds)[i];
        } else {
            for (int i = lt; i < bytes; i += nt) gmem[i] = lds[i];
        }
    }
}

// ------------------------------------------------------ resident items
namespace {

// The lanes of one replica meet: a barrier, or where a replica has at most a
// wave's lanes only an order of its LDS accesses (a wave's are served in order).
__device__ __forceinline__ void replica_sync(bool waves) {
    if (waves) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// Recorded sweeps of a replica: its lanes add their counts in LDS, kRecRows rows
// at a time, so that no sweep waits for a reduction or for global memory.
constexpr int kRecRows = 32;  // 6 KiB for kMaxRpb replicas, beside kResidentLdsBudget
struct RecRows {
    int (*l)[3];         // this replica's kRecRows x 3 counts in LDS
    int next, every;     // sweeps to the next recorded one
    int row0, n;         // first row and number of rows in LDS
    __device__ __forceinline__ void start(int (*lds)[3], const SweepArgs& a) {
        l = lds;
        every = a.record_every;
        next = every > 0 ? every - a.sweep_off % every : 0;
        row0 = every > 0 ? a.sweep_off / every : 0;
        n = 0;
    }
    // true at a recorded sweep
    __device__ __forceinline__ bool due() {
        if (every <= 0 || --next > 0) return false;
        next = every;
        return true;
    }
    // byte-wise counts; sums of 16 lanes (or of the 4 or 8 lanes of a replica: 64 lanes
    // hold at most 16) by data-parallel-primitive moves, then LDS atomics
    __device__ __forceinline__ void add(uint32_t up, uint32_t dx, uint32_t dy, int nt) {
        const int u = row_sum((int)sad_u8(up, 0u), nt);
        const int b = row_sum((int)(sad_u8(dx, 0u) | (sad_u8(dy, 0u) << 16)), nt);
        // lanes 0, 1, 2 of a group add one count each
        const int lane = (int)threadIdx.x & (min(nt, 16) - 1);
        const int v[3] = {u, b & 0xFFFF, (int)((uint32_t)b >> 16)};
        if (lane < 3) atomicAdd(&l[n][lane], lane == 0 ? v[0] : lane == 1 ? v[1] : v[2]);
    }
    // stores (SLAB: adds, the rows hold zeros or other slabs' shares) and clears
    // the rows; the replica's lanes meet before and after.  N: the sites counted.
    template <bool SLAB>
    __device__ __forceinline__ void flush(const SweepArgs& a, int rep, int N, bool active, int lt,
                                          int nt) {
        if (active)
            for (int i = lt; i < n * a.width; i += nt) {
                const int r = i / a.width, k = i - r * a.width;
                const int v = k < 3 ? l[r][k] : 0;
                const int share = k == 0 ? 2 * v - N : N - 2 * v;
                int32_t* at = a.stats + ((size_t)(row0 + r) * a.R + rep) * a.width + k;
                if (SLAB) {
                    if (k < 3) atomicAdd(at, share);
                } else {
                    *at = k < 3 ? share : 0;
                }
                if (k < 3) l[r][k] = 0;
            }
        row0 += n;
        n = 0;
    }
};

}  // namespace

// A workgroup owns a.rpb replicas of one shape for the whole call, blockDim /
// rpb = nt lanes each.  A lane owns NI items of a replica: 16 columns of two
// adjacent rows of both planes, in registers for the whole call; the planes in
// LDS carry them to the neighbours (two 16-byte and two 4-byte reads and two
// 16-byte writes an item and pass).  Everything that depends on the lane alone
// is computed once: a lane has one item in most shapes, and the index
// arithmetic of a pass used to cost as much as half a chunk.
// UNI: nt is a multiple of 64, so a wave's replica is uniform (scalar loads,
// Philox keys and counters in scalar registers).
// Bound by VALU operations where the chip is full (4096 lattices of 64 x 64, 100
// sweeps and 200 recorded ones: 2.59 -> 1.55 ms, 3.1e12 attempts/s), by one
// wave's latency for single small lattices.
template <int NI, bool UNI>
__global__ void __launch_bounds__(1024) k_resident_ising(SweepArgs a) {
    // dynamic LDS: rpb slots of [thresholds (kIsingTabWords) | plane 0 | plane 1]
    extern __shared__ __align__(16) uint8_t dyn[];
    __shared__ int lrec[kMaxRpb][kRecRows][3];  // counts of recorded sweeps
    const int P = a.rpb;
    const int nt = blockDim.x / P;
    int g = threadIdx.x / nt;
    const int lt = threadIdx.x - g * nt;
    if (UNI) g = __builtin_amdgcn_readfirstlane(g);
    const int first = blockIdx.x * P;
    const bool active = first + g < a.n_list;
    const int rep = a.rep_list[active ? first + g : first];
    const RepDev& R = a.reps[rep];
    const int W = R.W, Ly = R.Ly, cpr = W >> 4;
    const uint32_t plane = (uint32_t)(Ly * W), rid = R.rid;
    uint8_t* slot = dyn + (size_t)(active ? g : 0) * a.res_slot_bytes;
    uint32_t* tab = reinterpret_cast<uint32_t*>(slot);
    uint8_t* lds = slot + 4 * kIsingTabWords;
    uint8_t* gmem = a.lat + R.lat_off;
    const int n_items = active ? (Ly >> 1) * cpr : 0;
    if (active) load_ising_table(a.tab, R, tab, lt, nt);
    // per item: byte offset in a plane of the even row's chunk, of the rows
    // above it and below its odd row, and of the halo dwords of the even row
    uint32_t oo[NI], uo[NI], dof[NI], le[NI], re[NI];
    uint4 V[2][2][NI];  // [plane][row][item]
#pragma unroll
    for (int k = 0; k < NI; ++k) {
        const int it = lt + k * nt;
        const int r = it < n_items ? it / cpr : 0;
        const uint32_t j0 = it < n_items ? (uint32_t)(it - r * cpr) << 4 : 0u;
        const uint32_t ro = (uint32_t)(2 * r * W), last = plane - (uint32_t)W;
        oo[k] = ro + j0;
        uo[k] = (r == 0 ? last : ro - (uint32_t)W) + j0;
        dof[k] = (2 * r + 2 == Ly ? 0u : ro + 2u * (uint32_t)W) + j0;
        le[k] = ro + (j0 == 0u ? (uint32_t)W : j0) - 4u;
        re[k] = ro + (j0 + 16u == (uint32_t)W ? 0u : j0 + 16u);
        if (it < n_items) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    const uint32_t at = c * plane + oo[k] + (uint32_t)(o * W);
                    V[c][o][k] = *reinterpret_cast<const uint4*>(gmem + at);
                    *reinterpret_cast<uint4*>(lds + at) = V[c][o][k];
                }
        }
    }
    for (int i = threadIdx.x; i < 3 * kRecRows * P; i += blockDim.x) (&lrec[0][0][0])[i] = 0;
    __syncthreads();
    const bool waves = nt > 64;
    RecRows rr;
    rr.start(lrec[g], a);
    const uint64_t t0 = *a.t_base + (uint64_t)a.sweep_off;
    for (int i = 0; i < a.n_sweeps; ++i) {
        const uint64_t t = t0 + (uint64_t)i;
        const bool rec = rr.due();
        uint32_t up = 0u, dx = 0u, dy = 0u;  // this lane's counts of a recorded sweep
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const uint32_t p = (uint32_t)(2 * t + (uint64_t)c);
            uint8_t* own = lds + c * plane;
            const uint8_t* oth = lds + (1 - c) * plane;
#pragma unroll
            for (int k = 0; k < NI; ++k) {
                if (lt + k * nt >= n_items) continue;
                // even row: parity c; odd row: parity 1 - c (left halo for parity 0)
                const uint4 U = *reinterpret_cast<const uint4*>(oth + uo[k]);
                const uint4 D = *reinterpret_cast<const uint4*>(oth + dof[k]);
                const uint32_t e0 =
                    *reinterpret_cast<const uint32_t*>(oth + (c == 0 ? le[k] : re[k]));
                const uint32_t e1 =
                    *reinterpret_cast<const uint32_t*>(oth + W + (c == 0 ? re[k] : le[k]));
                uint32_t o0[4], o1[4], m0[4], m1[4], Uv[4], Dv[4], nv[4], sv[4];
                arr(V[c][0][k], o0);
                arr(V[c][1][k], o1);
                arr(V[1 - c][0][k], m0);
                arr(V[1 - c][1][k], m1);
                arr(U, Uv);
                arr(D, Dv);
                side_bytes(c, m0, e0, sv);
                ising_core(o0, m0, sv, Uv, m1, oo[k], p, rid, a.key0, a.key1, tab, nv);
                if (c == 1 && rec) ising_count(nv, m0, sv, Uv, m1, up, dx, dy);
                V[c][0][k] = make_uint4(nv[0], nv[1], nv[2], nv[3]);
                *reinterpret_cast<uint4*>(own + oo[k]) = V[c][0][k];
                side_bytes(1 - c, m1, e1, sv);
                ising_core(o1, m1, sv, m0, Dv, oo[k] + (uint32_t)W, p, rid, a.key0, a.key1, tab,
                           nv);
                if (c == 1 && rec) ising_count(nv, m1, sv, m0, Dv, up, dx, dy);
                V[c][1][k] = make_uint4(nv[0], nv[1], nv[2], nv[3]);
                *reinterpret_cast<uint4*>(own + oo[k] + W) = V[c][1][k];
            }
            if (c == 0) replica_sync(waves);
        }
        if (rec) {
            rr.add(up, dx, dy, nt);  // at most 16 NI a byte
            if (++rr.n == kRecRows) {
                replica_sync(waves);
                rr.flush<false>(a, rep, 2 * (int)plane, active, lt, nt);
            }
        }
        replica_sync(waves);
    }
    rr.flush<false>(a, rep, 2 * (int)plane, active, lt, nt);
#pragma unroll
    for (int k = 0; k < NI; ++k)
        if (lt + k * nt < n_items)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int o = 0; o < 2; ++o)
                    *reinterpret_cast<uint4*>(gmem + c * plane + oo[k] + (uint32_t)(o * W)) =
                        V[c][o][k];
}

namespace {

__device__ __forceinline__ uint32_t lds32(const uint8_t* p) {
    return *reinterpret_cast<const uint32_t*>(p);
}

// The first n bytes (even, at most 8) of v to a 2-byte aligned place.
__device__ __forceinline__ void put_bytes(uint8_t* p, const uint2& v, uint32_t n) {
    uint16_t* q = reinterpret_cast<uint16_t*>(p);
    if (n > 0u) q[0] = (uint16_t)v.x;
    if (n > 2u) q[1] = (uint16_t)(v.x >> 16);
    if (n > 4u) q[2] = (uint16_t)v.y;
    if (n > 6u) q[3] = (uint16_t)(v.y >> 16);
}

// A plane in LDS: stores an item (and, for item 0, the repeat behind the plane).
template <bool AL>
__device__ __forceinline__ void store8(uint8_t* own, uint32_t k, uint32_t plane, const uint2& v) {
    if (AL || (plane & 7u) == 0u) {
        *reinterpret_cast<uint2*>(own + k) = v;
        if (!AL && k == 0u) *reinterpret_cast<uint2*>(own + plane) = v;
    } else {
        if (k + 8u <= plane)
            *reinterpret_cast<uint2*>(own + k) = v;
        else
            put_bytes(own + k, v, plane - k);
        if (k == 0u) put_bytes(own + plane, v, 8u);
    }
}

// The other plane's neighbours of an item in colour c: side, above, below.
template <bool AL>
__device__ __forceinline__ void near8(const Item8<AL>& t, const uint8_t* oth, int c,
                                      const uint32_t (&m)[2], uint32_t (&sv)[2],
                                      uint32_t (&Uv)[2], uint32_t (&Dv)[2]) {
    if (AL) {
        const uint2 U = *reinterpret_cast<const uint2*>(oth + t.uo);
        const uint2 D = *reinterpret_cast<const uint2*>(oth + t.dof);
        const bool lf = (t.left[0] != 0u) == (c == 0);
        const uint32_t h = lds32(oth + (lf ? t.lo : t.hi));
        const uint32_t a0 = lf ? h : m[0], a1 = lf ? m[0] : m[1], a2 = lf ? m[1] : h;
        const uint32_t sh = lf ? 3u : 1u;
        sv[0] = __builtin_amdgcn_alignbyte(a1, a0, sh);
        sv[1] = __builtin_amdgcn_alignbyte(a2, a1, sh);
        Uv[0] = U.x;
        Uv[1] = U.y;
        Dv[0] = D.x;
        Dv[1] = D.y;
    } else {
        const uint8_t* u = oth + (t.uo & ~3u);
        const uint8_t* d = oth + (t.dof & ~3u);
        const uint32_t u0 = lds32(u), u1 = lds32(u + 4), u2 = lds32(u + 8);
        const uint32_t d0 = lds32(d), d1 = lds32(d + 4), d2 = lds32(d + 8);
        const uint32_t pv = lds32(oth + (t.k == 0u ? 0u : t.k - 4u)), nx = lds32(oth + t.k + 8u);
        const uint32_t eb = oth[t.hi] * 0x01010101u, sb = oth[t.lo] * 0x01010101u;
        Uv[0] = __builtin_amdgcn_alignbyte(u1, u0, t.uo);
        Uv[1] = __builtin_amdgcn_alignbyte(u2, u1, t.uo);
        Dv[0] = __builtin_amdgcn_alignbyte(d1, d0, t.dof);
        Dv[1] = __builtin_amdgcn_alignbyte(d2, d1, t.dof);
        const uint32_t L[2] = {__builtin_amdgcn_alignbyte(m[0], pv, 3),
                               __builtin_amdgcn_alignbyte(m[1], m[0], 3)};
        const uint32_t R[2] = {__builtin_amdgcn_alignbyte(m[1], m[0], 1),
                               __builtin_amdgcn_alignbyte(nx, m[1], 1)};
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t lf = c == 0 ? t.left[i] : ~t.left[i];
            const uint32_t fe = t.end[i] & ~lf, fs = t.start[i] & lf;
            uint32_t v = (lf & L[i]) | (~lf & R[i]);
            v = (fe & eb) | (~fe & v);
            sv[i] = (fs & sb) | (~fs & v);
        }
    }
}

// Both planes of a lattice between memory and LDS (with their repeats), by lanes
// lt = 0 .. nt - 1.
template <bool AL>
__device__ __forceinline__ void load_planes8(uint8_t* lds, const uint8_t* gmem, uint32_t plane,
                                             uint32_t stride, uint32_t lt, uint32_t nt) {
    if (AL || (plane & 7u) == 0u) {
        for (uint32_t k = 8u * lt; k < plane; k += 8u * nt)
#pragma unroll
            for (uint32_t c = 0; c < 2u; ++c)
                store8<AL>(lds + c * stride, k, plane,
                           *reinterpret_cast<const uint2*>(gmem + c * plane + k));
    } else {
        for (uint32_t i = lt; i < plane + 8u; i += nt)
#pragma unroll
            for (uint32_t c = 0; c < 2u; ++c)
                lds[c * stride + i] = gmem[c * plane + (i < plane ? i : i - plane)];
    }
}

template <bool AL>
__device__ __forceinline__ void store_planes8(uint8_t* gmem, const uint8_t* lds, uint32_t plane,
                                              uint32_t stride, uint32_t lt, uint32_t nt) {
    if (AL || (plane & 7u) == 0u) {
        for (uint32_t k = 8u * lt; k < plane; k += 8u * nt)
#pragma unroll
            for (uint32_t c = 0; c < 2u; ++c)
                *reinterpret_cast<uint2*>(gmem + c * plane + k) =
                    *reinterpret_cast<const uint2*>(lds + c * stride + k);
    } else {
        for (uint32_t i = lt; i < plane; i += nt)
#pragma unroll
            for (uint32_t c = 0; c < 2u; ++c) gmem[c * plane + i] = lds[c * stride + i];
    }
}

}  // namespace

// The resident kernel for items of eight sites: a lane takes one Philox block a
// pass instead of four, so a small lattice spreads over four times as many lanes
// and a pass is a quarter of the chain of instructions.  It serves lattices
// whose waves leave the chip idle (one 32 x 32 lattice, recorded: 0.8 us a sweep
// against 2.7) and, without AL, every other width from 18 on (k_resident_generic
// draws a block for every site: 100 lattices of 300 x 300, 20 sweeps and the
// gradients 2064 us, now 405).
// NI = 1, 2: at most NI items a lane, their offsets and both planes' bytes in
// registers; NI = 0: a lane's items are worked out in every pass.
//
// SLAB (with AL, NI > 0 and UNI): a few large lattices are cut into slabs of rows, a
// workgroup each, where whole ones would leave most of the chip idle.  A
// workgroup reads its slab with a.halo rows on either side from one of two lattices, runs
// n_sweeps <= a.halo / 2 sweeps on that window and writes its own rows to the other:
// the window's outermost valid row moves inwards by one a pass, since every
// site's draws depend on its place alone, so the slabs need no exchange between
// launches (64 lattices of 256 x 256: 2.7 us a sweep in slabs, 4.4 whole).
template <bool AL, int NI, bool UNI, bool SLAB>
__global__ void __launch_bounds__(1024) k_resident_ising8(SweepArgs a) {
    // dynamic LDS: rpb slots of [thresholds (kIsingTabWords) | plane 0 and its repeat |
    // plane 1 and its repeat], each plane in whole 8 bytes
    extern __shared__ __align__(16) uint8_t dyn[];
    __shared__ int lrec[kMaxRpb][kRecRows][3];
    const int P = a.rpb;
    const int nt = blockDim.x / P;
    int g = threadIdx.x / nt;
    const int lt = threadIdx.x - g * nt;
    if (UNI) g = __builtin_amdgcn_readfirstlane(g);
    const int first = blockIdx.x * P;
    const bool active = first + g < a.n_list;
    const TileDev T = SLAB ? a.tiles[blockIdx.x] : TileDev{};
    const int rep = SLAB ? T.rep : a.rep_list[active ? first + g : first];
    const RepDev& R = a.reps[rep];
    // the window: the whole lattice, or a slab and its halo rows
    const int rows = SLAB ? T.rows + 2 * a.halo : R.Ly;
    const uint32_t W = (uint32_t)R.W, plane = (uint32_t)rows * W, rid = R.rid;
    const uint32_t gplane = (uint32_t)R.Ly * W;
    const float inv = 1.0f / (float)W;
    const uint32_t stride = (plane + 15u) & ~7u;
    uint8_t* slot = dyn + (size_t)(active ? g : 0) * a.res_slot_bytes;
    uint32_t* tab = reinterpret_cast<uint32_t*>(slot);
    uint8_t* lds = slot + 4 * kIsingTabWords;
    uint8_t* gmem = a.lat + R.lat_off;
    const uint8_t* gsrc = gmem;
    if (SLAB) {
        uint8_t* g2 = a.lat2 + (size_t)T.lat2 * 256u;
        gsrc = a.from2 ? g2 : gmem;
        gmem = a.from2 ? gmem : g2;
    }
    // place in the lattice of a window's byte k
    auto place = [&](uint32_t k) {
        if (!SLAB) return k;
        const int at = (T.y0 - a.halo) * (int)W + (int)k;
        return (uint32_t)(at < 0 ? at + (int)gplane : at >= (int)gplane ? at - (int)gplane : at);
    };
    const uint32_t n_items = active ? (plane + 7u) >> 3 : 0u;
    if (active) load_ising_table(a.tab, R, tab, lt, nt);
    if (SLAB) {
        for (uint32_t i = lt; i < n_items; i += (uint32_t)nt)
#pragma unroll
            for (uint32_t c = 0; c < 2u; ++c)
                *reinterpret_cast<uint2*>(lds + c * stride + 8u * i) =
                    *reinterpret_cast<const uint2*>(gsrc + c * gplane + place(8u * i));
    } else if (active) {
        load_planes8<AL>(lds, gmem, plane, stride, (uint32_t)lt, (uint32_t)nt);
    }
    constexpr int NR = NI > 0 ? NI : 1;
    Item8<AL> it[NR];
    uint2 V[2][NR];
    uint32_t kb[NR];  // within-colour index
    int row[NR];      // SLAB: the window's row, -1 without an item
    auto held = [&](int n) { return (uint32_t)(lt + n * nt) < n_items; };
    // not a halo row
    auto mine = [&](int n) {
        return !SLAB || (row[n] >= a.halo && row[n] < a.halo + T.rows);
    };
    const int sites = SLAB ? 2 * T.rows * (int)W : 2 * (int)plane;  // counted here
    __syncthreads();
#pragma unroll
    for (int n = 0; n < NI; ++n) {
        it[n].init(held(n) ? (uint32_t)(lt + n * nt) : 0u, W, inv, plane);
        kb[n] = place(it[n].k);
        row[n] = SLAB ? (held(n) ? (int)(it[n].k / W) : -1) : 0;
#pragma unroll
        for (uint32_t c = 0; c < 2u; ++c)
            if (held(n)) V[c][n] = *reinterpret_cast<const uint2*>(lds + c * stride + it[n].k);
    }
    for (int i = threadIdx.x; i < 3 * kRecRows * P; i += blockDim.x) (&lrec[0][0][0])[i] = 0;
    __syncthreads();
    const bool waves = nt > 64;
    RecRows rr;
    rr.start(lrec[g], a);
    const uint64_t t0 = *a.t_base + (uint64_t)a.sweep_off;
    for (int sw = 0; sw < a.n_sweeps; ++sw) {
        const uint64_t t = t0 + (uint64_t)sw;
        const bool rec = rr.due();
        uint32_t up = 0u, dx = 0u, dy = 0u;  // this lane's counts of a recorded sweep
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const uint32_t p = (uint32_t)(2 * t + (uint64_t)c);
            uint8_t* own = lds + (uint32_t)c * stride;
            const uint8_t* oth = lds + (uint32_t)(1 - c) * stride;
            auto pass = [&](const Item8<AL>& q, uint32_t k0, bool cnt, uint2& o, const uint2& m2) {
                const uint32_t ov[2] = {o.x, o.y};
                uint32_t m[2] = {m2.x, m2.y}, sv[2], Uv[2], Dv[2], nv[2];
                near8<AL>(q, oth, c, m, sv, Uv, Dv);
                ising_core(ov, m, sv, Uv, Dv, k0, p, rid, a.key0, a.key1, tab, nv);
                o = make_uint2(nv[0], nv[1]);
                store8<AL>(own, q.k, plane, o);
                if (c == 1 && rec && cnt) {
                    if (!AL && q.k + 8u > plane) {
                        const uint64_t in = (1ull << (8u * (plane - q.k))) - 1ull;
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            const uint32_t w = (uint32_t)(in >> (32 * i));
                            nv[i] &= w;
                            m[i] &= w;
                            sv[i] &= w;
                            Uv[i] &= w;
                            Dv[i] &= w;
                        }
                    }
                    ising_count(nv, m, sv, Uv, Dv, up, dx, dy);
                }
            };
            if (NI > 0) {
                // after pass j the rows j + 1 .. rows - 2 - j are valid
                const int j = 2 * sw + c;
#pragma unroll
                for (int n = 0; n < NI; ++n)
                    if (SLAB ? row[n] > j && row[n] < rows - 1 - j : held(n))
                        pass(it[n], kb[n], mine(n), V[c][n], V[1 - c][n]);
            } else {
                for (uint32_t i = lt; i < n_items; i += (uint32_t)nt) {
                    Item8<AL> q;
                    q.init(i, W, inv, plane);
                    uint2 o = *reinterpret_cast<const uint2*>(own + q.k);
                    pass(q, q.k, true, o, *reinterpret_cast<const uint2*>(oth + q.k));
                }
            }
            if (c == 0) replica_sync(waves);
        }
        if (rec) {  // at most 4 a byte and item
            rr.add(up, dx, dy, nt);
            if (++rr.n == kRecRows) {
                replica_sync(waves);
                rr.flush<SLAB>(a, rep, sites, active, lt, nt);
            }
        }
        replica_sync(waves);
    }
    rr.flush<SLAB>(a, rep, sites, active, lt, nt);
    if (SLAB) {
#pragma unroll
        for (int n = 0; n < NI; ++n)
            if (mine(n))
#pragma unroll
                for (uint32_t c = 0; c < 2u; ++c)
                    *reinterpret_cast<uint2*>(gmem + c * gplane + kb[n]) = V[c][n];
    } else if (active) {
        store_planes8<AL>(gmem, lds, plane, stride, (uint32_t)lt, (uint32_t)nt);
    }
}

// A recorded sweep of a replica: adds the lanes' counts (labels of q > 8 are in
// lhist already) to its row in LDS, (Nx, Ny, S, the most frequent label's count),
// and clears lhist.  The replica's lanes meet in it, and meet again before lhist
// or the row is next used.
__device__ __forceinline__ void potts_record(const PottsAcc& pa, int q, int lt, int nt, int* lhist,
                                             int* row) {
    add_counts<true>(pa, q, nt, lhist, row);
    replica_sync(nt > 64);
    if (q <= 8 && nt >= 8) {
        int mx = 0;
        if (lt < 8) {
            mx = lhist[lt];
            lhist[lt] = 0;
        }
        mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0xB1, 0xf, 0xf, true));
        mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0x4E, 0xf, 0xf, true));
        mx = max(mx, __builtin_amdgcn_update_dpp(0, mx, 0x141, 0xf, 0xf, true));
        if (lt == 0) row[3] = mx;
    } else if (lt < q) {
        int mx = 0;
        for (int k = lt; k < q; k += nt) {
            mx = max(mx, lhist[k]);
            lhist[k] = 0;
        }
        int at = 3;
        asm volatile("" : "+v"(at));  // a plain atomic, not a reduction over the wave first
        atomicMax(&row[at], mx);
    }
}

// Stores and clears the n rows behind row0.
__device__ __forceinline__ void potts_flush(const SweepArgs& a, int rep, int row0, int n,
                                            bool active, int lt, int nt, int (*rows)[4]) {
    if (!active) return;
    for (int i = lt; i < n * a.width; i += nt) {
        const int r = i / a.width, k = i - r * a.width;
        a.stats[((size_t)(row0 + r) * a.R + rep) * a.width + k] = k < 4 ? rows[r][k] : 0;
        if (k < 4) rows[r][k] = 0;
    }
}

// Resident Potts lattices by items of eight sites, two Philox blocks a lane and
// pass, for every width from 16 on (AL, NI, UNI as for k_resident_ising8, NI = 0
// or 1).  Bound by VALU operations (about 27 slots a site in lattices of three-bit
// labels without a field) or by a wave's latency: 1024 lattices of 64 x 64 take 1.9 us
// a pass (3.6 by chunks of 16 sites) and 3.0 with every sweep recorded (12.5 when
// that read every site with its neighbours).
template <bool AL, int NI, bool UNI>
__global__ void __launch_bounds__(1024) k_resident_potts8(SweepArgs a) {
    // dynamic LDS: rpb slots of [thresholds (tab_lds_bytes) | plane 0 and its repeat |
    // plane 1 and its repeat]
    extern __shared__ __align__(16) uint8_t dyn[];
    __shared__ int lhist[kMaxRpb][kMaxPottsQ];
    __shared__ int lrow[kMaxRpb][kPottsRecRows][4];
    static_assert(sizeof lhist + sizeof lrow == kPottsStaticLds, "LDS budget");
    const int P = a.rpb;
    const int nt = blockDim.x / P;
    int g = threadIdx.x / nt;
    const int lt = threadIdx.x - g * nt;
    if (UNI) g = __builtin_amdgcn_readfirstlane(g);
    const int first = blockIdx.x * P;
    const bool active = first + g < a.n_list;
    const int rep = a.rep_list[active ? first + g : first];
    const RepDev& R = a.reps[rep];
    const uint32_t W = (uint32_t)R.W, plane = (uint32_t)R.Ly * W, rid = R.rid;
    const uint32_t stride = (plane + 15u) & ~7u;
    const float inv = 1.0f / (float)W;
    const int q = R.q, ntab = R.tab_n, path = potts_path(R);
    const uint32_t lem = lemire_threshold(q);
    uint8_t* slot = dyn + (size_t)(active ? g : 0) * a.res_slot_bytes;
    uint32_t* tab = reinterpret_cast<uint32_t*>(slot);
    uint8_t* lds = slot + a.tab_lds_bytes;
    uint8_t* gmem = a.lat + R.lat_off;
    const uint32_t n_items = active ? (plane + 7u) >> 3 : 0u;
    if (active) {
        load_potts_table(a.tab, R, tab, lt, nt);
        load_planes8<AL>(lds, gmem, plane, stride, (uint32_t)lt, (uint32_t)nt);
    }
    for (int i = threadIdx.x; i < P * kMaxPottsQ; i += blockDim.x) (&lhist[0][0])[i] = 0;
    for (int i = threadIdx.x; i < P * kPottsRecRows * 4; i += blockDim.x) (&lrow[0][0][0])[i] = 0;
    __syncthreads();
    Item8<AL> it;
    const bool held = NI > 0 && (uint32_t)lt < n_items;
    uint2 vo, vm;  // NI = 1: the item's bytes in the colour at work and in the other
    if (NI > 0) {
        it.init(held ? (uint32_t)lt : 0u, W, inv, plane);
        vo = *reinterpret_cast<const uint2*>(lds + it.k);
        vm = *reinterpret_cast<const uint2*>(lds + stride + it.k);
    }
    const bool waves = nt > 64;
    const uint64_t t0 = *a.t_base + (uint64_t)a.sweep_off;
    int next = a.record_every > 0 ? a.record_every - a.sweep_off % a.record_every : 0;
    int row0 = a.record_every > 0 ? a.sweep_off / a.record_every : 0, n_rows = 0;
    for (int sw = 0; sw < a.n_sweeps; ++sw) {
        const uint64_t t = t0 + (uint64_t)sw;
        bool rec = false;
        if (a.record_every > 0 && --next == 0) {
            next = a.record_every;
            rec = true;
        }
        PottsAcc pa;
        pa.clear();
#pragma nounroll
        for (int c = 0; c < 2; ++c) {
            const uint32_t p = (uint32_t)(2 * t + (uint64_t)c);
            uint8_t* own = lds + (uint32_t)c * stride;
            const uint8_t* oth = lds + (uint32_t)(1 - c) * stride;
            auto pass = [&](const Item8<AL>& e, uint2& o, const uint2& m2) {
                const uint32_t ov[2] = {o.x, o.y}, m[2] = {m2.x, m2.y};
                uint32_t sv[2], Uv[2], Dv[2], nv[2];
                near8<AL>(e, oth, c, m, sv, Uv, Dv);
                if (path == kPottsFast)
                    potts_core<2, kPottsFast>(ov, m, sv, Uv, Dv, e.k, p, rid, a.key0, a.key1, tab,
                                              q, ntab, lem, nv);
                else if (path == kPottsNoField)
                    potts_core<2, kPottsNoField>(ov, m, sv, Uv, Dv, e.k, p, rid, a.key0, a.key1,
                                                 tab, q, ntab, lem, nv);
                else
                    potts_core<2, kPottsAny>(ov, m, sv, Uv, Dv, e.k, p, rid, a.key0, a.key1, tab,
                                             q, ntab, lem, nv);
                o = make_uint2(nv[0], nv[1]);
                store8<AL>(own, e.k, plane, o);
                if (c == 1 && rec) {
                    if (AL || e.k + 8u <= plane) {
                        potts_count(nv, m, sv, Uv, Dv, q, pa, lhist[g]);
                    } else {  // the last item's sites
                        for (uint32_t j = 0; j < plane - e.k; ++j) {
                            const uint32_t sh = 8u * (j & 3u);
                            auto at = [&](const uint32_t (&v)[2]) {
                                return ((j < 4u ? v[0] : v[1]) >> sh) & 0xFFu;
                            };
                            const uint32_t s = at(nv), x = at(m);
                            pa.Nx += (s == x) + (s == at(sv));
                            pa.Ny += (s == at(Uv)) + (s == at(Dv));
                            pa.S += (int)(s + x);
                            atomicAdd(&lhist[g][s], 1);
                            atomicAdd(&lhist[g][x], 1);
                        }
                    }
                }
            };
            if (NI > 0) {
                if (held) pass(it, vo, vm);
                const uint2 v = vo;
                vo = vm;
                vm = v;
            } else {
                for (uint32_t i = lt; i < n_items; i += (uint32_t)nt) {
                    Item8<AL> e;
                    e.init(i, W, inv, plane);
                    uint2 o = *reinterpret_cast<const uint2*>(own + e.k);
                    pass(e, o, *reinterpret_cast<const uint2*>(oth + e.k));
                }
            }
            if (c == 0) replica_sync(waves);
        }
        if (rec) {
            potts_record(pa, q, lt, nt, lhist[g], lrow[g][n_rows]);
            if (++n_rows == kPottsRecRows) {
                replica_sync(waves);
                potts_flush(a, rep, row0, n_rows, active, lt, nt, lrow[g]);
                row0 += n_rows;
                n_rows = 0;
            }
        }
        replica_sync(waves);
    }
    potts_flush(a, rep, row0, n_rows, active, lt, nt, lrow[g]);
    if (active) store_planes8<AL>(gmem, lds, plane, stride, (uint32_t)lt, (uint32_t)nt);
}

__global__ void k_init(const RepDev* reps, const int32_t* list, uint8_t* lat, uint32_t k0,
                       uint32_t k1) {
    const RepDev R = reps[list[blockIdx.y]];
    const int N = R.Lx * R.Ly;
    uint8_t* planes = lat + R.lat_off;
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; 4 * b < N; b += gridDim.x * blockDim.x) {
        uint32_t w[4];
        philox4x32_10((uint32_t)b, 0u, R.rid, kTagInit, k0, k1, w);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int n = 4 * b + i;
            if (n >= N) break;
            const int y = n / R.Lx, x = n - y * R.Lx;
            uint8_t v;
            if (R.model == kModelIsing)
                v = (w[i] < 0x80000000u) ? 1 : 0;
            else
                v = (uint8_t)(((uint64_t)w[i] * (uint64_t)R.q) >> 32);
            planes[(size_t)((x + y) & 1) * R.Ly * R.W + (size_t)y * R.W + (x >> 1)] = v;
        }
    }
}

// Statistics of every lattice, grid (parts of a lattice, replicas).  Rows of whole 16-site chunks count as a recorded
// colour-1 pass does, other widths site by site; Potts labels gather in LDS (one
// atomic a site in memory took 9 ms for 512 lattices of up to 1024 x 1024, now
// about 100 us).
__global__ void __launch_bounds__(256) k_measure(const RepDev* reps, const int32_t* list,
                                                 const uint8_t* lat, int32_t* stats, int32_t* hist,
                                                 int width) {
    __shared__ int lred[64];
    __shared__ int lhist[kMaxPottsQ];
    const int r = list[blockIdx.y];
    const RepDev R = reps[r];
    const uint8_t* p0 = lat + R.lat_off;
    const bool potts = R.model == kModelPotts;
    const int n_items = (R.W & 15) == 0 ? (R.Ly >> 1) * (R.W >> 4) : R.Lx * R.Ly;
    if ((int)(blockIdx.x * blockDim.x) >= n_items) return;
    for (int i = threadIdx.x; i < kMaxPottsQ; i += blockDim.x) lhist[i] = 0;
    __syncthreads();
    PottsAcc pa;
    pa.clear();
    int v[3] = {0, 0, 0};
    const int stride = gridDim.x * blockDim.x;
    if ((R.W & 15) == 0) {
        const uint32_t W = (uint32_t)R.W, last = (uint32_t)(R.Ly - 1) * W, cpr = W >> 4;
        const uint8_t* p1 = p0 + (size_t)R.Ly * W;
#pragma unroll
        for (int par = 0; par < 2; ++par)  // rows of parity (y + 1) & 1 = par
            for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_items; i += stride) {
                const uint32_t y = (uint32_t)i / cpr, j0 = ((uint32_t)i - y * cpr) << 4;
                const uint32_t ro = (2u * y + (par ? 0u : 1u)) * W;
                ChunkIn in;
                if (par == 0) {
                    const ChunkOff<0> f(ro, j0, W, last);
                    in = chunk_load<false>(p1, p0, f.oo, f.uo, f.dof, f.eo);
                } else {
                    const ChunkOff<1> f(ro, j0, W, last);
                    in = chunk_load<false>(p1, p0, f.oo, f.uo, f.dof, f.eo);
                }
                uint32_t ov[4], mv[4], Uv[4], Dv[4], sv[4];
                arr(in.o, ov);
                arr(in.m, mv);
                arr(in.U, Uv);
                arr(in.D, Dv);
                side_bytes(par, mv, in.e, sv);
                if (potts) {
                    potts_count(ov, mv, sv, Uv, Dv, R.q, pa, lhist);
                } else {
                    uint32_t up = 0u, dx = 0u, dy = 0u;
                    ising_count(ov, mv, sv, Uv, Dv, up, dx, dy);
                    v[0] += 2 * (int)sad_u8(up, 0u) - 32;
                    v[1] += 32 - 2 * (int)sad_u8(dx, 0u);
                    v[2] += 32 - 2 * (int)sad_u8(dy, 0u);
                }
            }
        if (potts) {
            v[0] = pa.Nx;
            v[1] = pa.Ny;
            v[2] = pa.S;
            if (R.q <= 8) add_counts<false>(pa, R.q, 64, lhist, nullptr);
        }
    } else {
        for (int n0 = blockIdx.x * blockDim.x; n0 < n_items; n0 += stride)
            lattice_stats(R.model, p0, R.Lx, R.Ly, R.W, n0, min(n_items, n0 + (int)blockDim.x), v,
                          lhist);
    }
    block_sum<3>(v, lred);  // its barriers order the labels too
    if (threadIdx.x == 0) {
        atomicAdd(&stats[(size_t)r * width + 0], v[0]);
        atomicAdd(&stats[(size_t)r * width + 1], v[1]);
        atomicAdd(&stats[(size_t)r * width + 2], v[2]);
    }
    if (potts)
        for (int i = threadIdx.x; i < R.q; i += blockDim.x)
            if (lhist[i]) atomicAdd(&hist[R.hist_off + i], lhist[i]);
}

__global__ void k_fill_i32(int32_t* p, size_t n, int32_t v) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_advance(uint64_t* t, uint64_t n) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *t += n;
}

__global__ void k_copy_counter(uint64_t* t) {
    if (threadIdx.x == 0 && blockIdx.x == 0) t[1] = t[0];
}

// FP64 observables from integer statistics (one thread per replica).
__global__ void k_observables(const RepDev* reps, int R, const int32_t* stats, int width,
                              double* obs) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= R) return;
    const RepDev D = reps[r];
    const int32_t* s = stats + (size_t)r * width;
    const double N = (double)D.Lx * (double)D.Ly;
    double* o = obs + (size_t)r * 4;
    if (D.model == kModelIsing) {
        const double M = s[0], Bx = s[1], By = s[2];
        const double H = -((double)D.Jx * Bx + (double)D.Jy * By + (double)D.h * M);
        o[0] = H / N;
        o[1] = fabs(M) / N;
        o[2] = (M / N) * (M / N);
        o[3] = M / N;
    } else if (D.model == kModelPotts) {
        const double Nx = s[0], Ny = s[1], S = s[2], nm = s[3];
        const double H = -((double)D.Jx * (Nx + Ny) + (double)D.h * S);
        o[0] = H / N;
        o[1] = ((double)D.q * nm / N - 1.0) / ((double)D.q - 1.0);
        o[2] = S / N;
        o[3] = 0.0;
    } else {
        const uint64_t lo = (uint32_t)s[10], hi = (uint32_t)s[11];
        const int64_t H = (int64_t)((hi << 32) | lo);
        o[0] = (double)H / (double)D.S;
        o[1] = 0.0;
        o[2] = 0.0;
        o[3] = 0.0;
    }
}

// ---------------------------------------------------------------- launchers
hipError_t launch_init(const RepDev* reps, const int32_t* list, int n, uint8_t* lat,
                       uint32_t key0, uint32_t key1, int threads, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    dim3 grid(64, n);
    hipLaunchKernelGGL(k_init, grid, dim3(threads), 0, s, reps, list, lat, key0, key1);
    return hipGetLastError();
}

namespace {
template <bool AL, bool UNI>
const void* ising8_fn(int items, int nt) {
    return items <= nt       ? (const void*)k_resident_ising8<AL, 1, UNI, false>
           : items <= 2 * nt ? (const void*)k_resident_ising8<AL, 2, UNI, false>
                             : (const void*)k_resident_ising8<AL, 0, UNI, false>;
}

template <bool AL, bool UNI>
const void* potts8_fn(int items, int nt) {
    return items <= nt ? (const void*)k_resident_potts8<AL, 1, UNI>
                       : (const void*)k_resident_potts8<AL, 0, UNI>;
}

const void* resident_fn(int kind, int items, int nt) {
    const bool uni = nt % 64 == 0;
    switch (kind) {
        case kResIsing16:
            return items > nt ? (uni ? (const void*)k_resident_ising<2, true>
                                     : (const void*)k_resident_ising<2, false>)
                              : (uni ? (const void*)k_resident_ising<1, true>
                                     : (const void*)k_resident_ising<1, false>);
        case kResIsing8: return uni ? ising8_fn<true, true>(items, nt) : ising8_fn<true, false>(items, nt);
        case kResIsing8Any:
            return uni ? ising8_fn<false, true>(items, nt) : ising8_fn<false, false>(items, nt);
        case kResIsingSlab:
            return items <= nt ? (const void*)k_resident_ising8<true, 1, true, true>
                               : (const void*)k_resident_ising8<true, 2, true, true>;
        case kResPotts8: return uni ? potts8_fn<true, true>(items, nt) : potts8_fn<true, false>(items, nt);
        case kResPotts8Any:
            return uni ? potts8_fn<false, true>(items, nt) : potts8_fn<false, false>(items, nt);
        default: return (const void*)k_resident_generic;
    }
}
}  // namespace

hipError_t resident_reserve_lds(int kind, int items, int nt, size_t lds_bytes) {
    return hipFuncSetAttribute(resident_fn(kind, items, nt),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
}

hipError_t launch_resident(const SweepArgs& a, int n_list, int kind, int items, int threads,
                           size_t lds_bytes, hipStream_t s) {
    if (n_list <= 0) return hipSuccess;
    const int nt = threads / a.rpb;
    if ((kind == kResIsing16 || kind == kResIsingSlab) && items > 2 * nt) return hipErrorInvalidValue;
    SweepArgs b = a;
    void* args[] = {&b};
    return hipLaunchKernel(resident_fn(kind, items, nt), dim3((n_list + a.rpb - 1) / a.rpb),
                           dim3(threads), args, lds_bytes, s);
}

hipError_t launch_stream_pass(const SweepArgs& a, int model, int tile0, int n_tiles, int c,
                              int sweep_off, int rec_row, int threads, size_t lds_tab_bytes,
                              bool nt, hipStream_t s) {
    if (n_tiles <= 0) return hipSuccess;
    const dim3 g(n_tiles), b(threads);
    if (model == kModelIsing) {
        if (nt)
            hipLaunchKernelGGL(k_stream_pass_ising<true>, g, b, 0, s, a, tile0, n_tiles, c,
                               sweep_off, rec_row);
        else
            hipLaunchKernelGGL(k_stream_pass_ising<false>, g, b, 0, s, a, tile0, n_tiles, c,
                               sweep_off, rec_row);
    } else {
        if (nt)
            hipLaunchKernelGGL(k_stream_pass_potts<true>, g, b, lds_tab_bytes, s, a, tile0, n_tiles,
                               c, sweep_off, rec_row);
        else
            hipLaunchKernelGGL(k_stream_pass_potts<false>, g, b, lds_tab_bytes, s, a, tile0,
                               n_tiles, c, sweep_off, rec_row);
    }
    return hipGetLastError();
}

namespace {
const void* persist_fn(int model, bool nt) {
    if (model == kModelIsing)
        return nt ? (const void*)k_persist_ising<true> : (const void*)k_persist_ising<false>;
    return nt ? (const void*)k_persist_potts<true> : (const void*)k_persist_potts<false>;
}
}  // namespace

hipError_t persist_reserve_lds(size_t lds_bytes) {
    hipError_t e = hipSuccess;
    for (int m = 0; m < 2 && e == hipSuccess; ++m)
        for (int nt = 0; nt < 2 && e == hipSuccess; ++nt)
            e = hipFuncSetAttribute(persist_fn(m, nt != 0),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    return e;
}

hipError_t persist_occupancy(int model, bool nt, size_t lds_bytes, int* per_cu) {
    *per_cu = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, persist_fn(model, nt), 256,
                                                        lds_bytes);
}

hipError_t launch_persist(const SweepArgs& a, int model, const PersistItem* items,
                          const int32_t* item_off, int n_wg, uint32_t* flags, uint32_t* abort_flag,
                          int slot_words, size_t lds_bytes, bool nt, hipStream_t s) {
    if (n_wg <= 0) return hipSuccess;
    const dim3 g(n_wg), b(256);
    if (model == kModelIsing) {
        if (nt)
            hipLaunchKernelGGL(k_persist_ising<true>, g, b, lds_bytes, s, a, items, item_off, flags,
                               abort_flag, slot_words);
        else
            hipLaunchKernelGGL(k_persist_ising<false>, g, b, lds_bytes, s, a, items, item_off,
                               flags, abort_flag, slot_words);
    } else {
        if (nt)
            hipLaunchKernelGGL(k_persist_potts<true>, g, b, lds_bytes, s, a, items, item_off, flags,
                               abort_flag, slot_words);
        else
            hipLaunchKernelGGL(k_persist_potts<false>, g, b, lds_bytes, s, a, items, item_off,
                               flags, abort_flag, slot_words);
    }
    return hipGetLastError();
}

hipError_t launch_potts_hist_finalize(const SweepArgs& a, const int32_t* list, int n, int rec_row,
                                      hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_potts_hist_finalize, dim3((n + 255) / 256), dim3(256), 0, s, a, list, n,
                       rec_row);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* p, size_t n, int32_t v, hipStream_t s) {
    if (n == 0) return hipSuccess;
    size_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_copy_counter(uint64_t* t, hipStream_t s) {
    hipLaunchKernelGGL(k_copy_counter, dim3(1), dim3(64), 0, s, t);
    return hipGetLastError();
}

hipError_t launch_advance(uint64_t* t, uint64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, s, t, n);
    return hipGetLastError();
}

hipError_t launch_measure(const RepDev* reps, const int32_t* list, int n, int max_sites,
                          const uint8_t* lat, int32_t* stats, int32_t* hist, int width,
                          hipStream_t s) {
    if (n <= 0) return hipSuccess;
    // about 16384 sites a workgroup, at most 64 workgroups a replica; those past a
    // smaller replica's items exit
    const int gx = std::min(64, (max_sites + 16383) / 16384);
    hipLaunchKernelGGL(k_measure, dim3(gx, n), dim3(256), 0, s, reps, list, lat, stats, hist,
                       width);
    return hipGetLastError();
}

hipError_t launch_observables(const RepDev* reps, int R, const int32_t* stats, int width,
                              double* obs, hipStream_t s) {
    hipLaunchKernelGGL(k_observables, dim3((R + 127) / 128), dim3(128), 0, s, reps, R, stats,
                       width, obs);
    return hipGetLastError();
}

}  // namespace spinmc
