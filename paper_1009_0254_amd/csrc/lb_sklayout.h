// Layout of the structure-factor sampler's row spectra (private to the library).
#pragma once

#include <hip/hip_runtime.h>

namespace lbf {

// One mode's row spectrum of a replica is stored in chunks of KG adjacent kx: [chunk][ky][KG]
// complex values of ELEM bytes, so that the column pass reads each chunk's rows as one contiguous run (a
// plain [ky][nh] layout puts consecutive ky of one kx a row apart and every read in another
// HBM page).  nh = nx/2 + 1 is padded to a multiple of KG.
// KG: 8 in FP32 (us per sample, 8 / 16: 4096^2 906 / 950, 2048^2 218 / 233, 256 x 16384 257 / 317), 16 in FP64
// (256 x 16384 565 / 555; 4096^2 1723 / 1718, 2048^2 388 / 388).
constexpr int sk_kg(int elem) { return elem == 8 ? 8 : 16; }
__host__ __device__ inline long long sk_nh_padded(int nx, int elem)
{
    const int kg = sk_kg(elem);
    return (long long)((nx / 2 + kg) / kg) * kg;
}
template <int ELEM> __device__ inline long long sk_at(int ky, int kx, int ny)
{
    constexpr int KG = sk_kg(ELEM);
    return ((long long)(kx / KG) * ny + ky) * KG + (kx % KG);
}
// the same in 32-bit arithmetic (one replica's mode slot holds fewer than 2^32 elements)
template <int ELEM> __device__ inline unsigned sk_at32(int ky, int kx, int ny)
{
    constexpr unsigned KG = sk_kg(ELEM);
    return (((unsigned)kx / KG) * (unsigned)ny + (unsigned)ky) * KG + ((unsigned)kx % KG);
}

}  // namespace lbf
