// Index of the network's upsampling (k_up2), apart so that the host can check it at sizes
// that no test allocates.
#pragma once

#if defined(__HIPCC__)
#define ERT_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define ERT_HOST_DEVICE inline
#endif

namespace ertvie {

// Fine voxel v = (x, y, z) and first of the four channels of one thread.  32 unsigned bits:
// a launch has fewer than 2^32 threads per dimension (HIP refuses more), a signed index
// would end at half of that.  Threads past the grid have z >= n2.
struct Up2Cell {
    unsigned v, x, y, z, c;
};

ERT_HOST_DEVICE Up2Cell up2_cell(unsigned block, unsigned threads, unsigned thread, unsigned C, unsigned n0, unsigned n1)
{
    const unsigned i = block * threads + thread, C4 = C / 4;
    Up2Cell q;
    q.v = i / C4;
    q.c = 4 * (i - q.v * C4);
    const unsigned r = q.v / n0;
    q.x = q.v - r * n0;
    q.y = r % n1;
    q.z = r / n1;
    return q;
}

}  // namespace ertvie
