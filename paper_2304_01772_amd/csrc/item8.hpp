// Offsets of a lane's eight sites in the colour planes of a resident lattice (plain
// arithmetic, so that a host program can check every one against the planes' size).
#pragma once
#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#else
#define __device__
#define __forceinline__ inline
inline unsigned __umul24(unsigned a, unsigned b) { return (a & 0xFFFFFFu) * (b & 0xFFFFFFu); }
#endif
#include <stdint.h>

namespace spinmc {

// Eight consecutive sites of a plane, one Philox block, from byte k on.  With AL
// (W a multiple of 8) they lie in one row; without, they may run on into the
// next one (W >= 9): e is the byte that ends a row, s the byte that starts one.
// Offsets wrap around the plane; a plane's first 8 bytes are repeated behind it.
// The last item may hold fewer sites (Ly W is even): its further bytes are 0 or 1,
// updated like the others, never stored or counted.
template <bool AL>
struct Item8 {
    uint32_t k, uo, dof;   // this item, the sites above and below
    uint32_t lo, hi;       // AL: halo dwords left and right; else: bytes ending the row that
                           // starts here and starting the row that ends here
    uint32_t left[2];      // bytes whose side neighbour is the left one in colour 0
    uint32_t end[2], start[2];  // !AL: the bytes e and s
    // inv = 1 / W: k <= 2^16 and W >= 8, so (k + 1/2) inv is off by less than its
    // distance from a whole number, 1 / (2 W)
    __device__ __forceinline__ void init(uint32_t item, uint32_t W, float inv, uint32_t plane) {
        k = 8u * item;
        const uint32_t y = (uint32_t)(((float)k + 0.5f) * inv), j = k - __umul24(y, W);
        const uint32_t row = k - j;
        uo = k < W ? k + plane - W : k - W;
        dof = k + W >= plane ? k + W - plane : k + W;
        if (AL) {
            left[0] = (y & 1u) ? 0u : ~0u;
            lo = row + (j == 0u ? W : j) - 4u;
            hi = row + (j + 8u == W ? 0u : j + 8u);
        } else {
            const uint32_t b = W - j;  // bytes of row y from here on
            const uint64_t first = b >= 8u ? ~0ull : (1ull << (8u * b)) - 1ull;
            const uint64_t lm = (y & 1u) ? ~first : first;
            const uint64_t em = b <= 8u ? 0xFFull << (8u * (b - 1u)) : 0ull;
            const uint64_t sm = j == 0u ? 0xFFull : (b < 8u ? 0xFFull << (8u * b) : 0ull);
            left[0] = (uint32_t)lm;
            left[1] = (uint32_t)(lm >> 32);
            end[0] = (uint32_t)em;
            end[1] = (uint32_t)(em >> 32);
            start[0] = (uint32_t)sm;
            start[1] = (uint32_t)(sm >> 32);
            hi = row;
            // (in the last row there is no next one: any byte of the plane will do)
            lo = j == 0u ? row + W - 1u : (b < 8u && row + W < plane ? row + 2u * W - 1u : row);
        }
    }
};

}  // namespace spinmc
