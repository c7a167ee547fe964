// Addresses of the tile copies global -> LDS, for the kernels and, compiled for the CPU, for the test of their bounds.
// Tiles lie in LDS row by row, the 16-byte chunks of a row swizzled: K^ a row per key of D bytes, V^ a row per channel of 128 bytes.
#pragma once
#if defined(__HIP__)
#define SAGE_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define SAGE_HOST_DEVICE inline
#endif

namespace sage {

template <int D>
SAGE_HOST_DEVICE constexpr int k_swz(int row) {
    return D == 128 ? (row & 7) : ((row >> 1) & 3);
}
// where chunk c16 of a row lies in the tile
template <int D>
SAGE_HOST_DEVICE constexpr int k_off(int row, int c16) {
    return row * D + ((c16 ^ k_swz<D>(row)) << 4);
}
SAGE_HOST_DEVICE constexpr int v_off(int row, int c16) { return row * 128 + ((c16 ^ (row & 7)) << 4); }

// The source offset, from the first byte of a tile (or of a piece of whole swizzle periods), of the chunk that a copy puts at 16 * slot:
// the swizzle is its own inverse.
template <int D>
SAGE_HOST_DEVICE constexpr int k_source(unsigned slot) {
    return k_off<D>((int)(slot / (D / 16)), (int)(slot % (D / 16)));
}
SAGE_HOST_DEVICE constexpr int v_source(unsigned slot) { return v_off((int)(slot >> 3), (int)(slot & 7)); }

// The size that a copy's descriptor gets: what is left of the head's buffer from its base on (chunks behind it are not fetched).
SAGE_HOST_DEVICE constexpr int copy_left(int head_bytes, int first) { return head_bytes - first > 0 ? head_bytes - first : 0; }

// decode_kernel: half tile `part` of key step j (K^: 64 keys, V^: half the channels) begins here; its piece p of 1 KB is at + 1024 p.
template <int D>
SAGE_HOST_DEVICE constexpr int half_first(int j, int part) {
    return (j * 2 + (part & 1)) * 64 * D;
}

}  // namespace sage
