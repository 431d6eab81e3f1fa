// mp_krylov.h -- sums of the single-workgroup Krylov solves (coarsest grids).
#pragma once
#include "mp_device.h"

namespace mp {

constexpr int kWaves = 16;  // wavefronts the sums are grouped by

// a in the lower half (of the wavefront, or of each pair of rows) and b in the
// upper one, each added to its value of the other half.
template <bool ROWS>
__device__ __forceinline__ double fold2(double a, double b)
{
    const unsigned long long ua = __builtin_bit_cast(unsigned long long, a);
    const unsigned long long ub = __builtin_bit_cast(unsigned long long, b);
    const unsigned al = (unsigned)ua, ah = (unsigned)(ua >> 32), bl = (unsigned)ub, bh = (unsigned)(ub >> 32);
    const auto lo = ROWS ? __builtin_amdgcn_permlane16_swap(al, bl, false, false)
                         : __builtin_amdgcn_permlane32_swap(al, bl, false, false);
    const auto hi = ROWS ? __builtin_amdgcn_permlane16_swap(ah, bh, false, false)
                         : __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}

// v[0..VJ) each added over the 64 lanes in the association of wave_sum, all in
// one go: lanes 64 / VJ * j and up end with the total of v[j].
template <int VJ>
__device__ __forceinline__ double wave_sums(const double (&v)[VJ])
{
    double s;
    if constexpr (VJ == 4) s = fold2<true>(fold2<false>(v[0], v[2]), fold2<false>(v[1], v[3]));
    else if constexpr (VJ == 2) s = swap_add<true>(fold2<false>(v[0], v[1]));
    else return wave_sum(v[0]);
    s = dpp_add<0x128>(s);
    s = dpp_add<0x124>(s);
    s = dpp_add<0x4e>(s);
    return dpp_add<0xb1>(s);
}

// Block sums of NV values in 1024 / VJ threads, each thread standing for VJ of
// 1024: v[a][j] belongs to wavefront (threadIdx.x / 64) + 16 / VJ * j of
// sixteen, and the sixteen totals are added in order, as block_sum does in 1024
// threads.  One barrier: the totals go to one half of `red`, and the halves
// alternate, so the next call's writes never meet this call's reads.
template <int VJ, int NV>
__device__ __forceinline__ void totals(const double (&v)[NV][VJ], double (&out)[NV], double (*red)[2][kWaves], int& half)
{
#pragma unroll
    for (int a = 0; a < NV; a++) {
        const double s = wave_sums<VJ>(v[a]);
        const int l = (int)threadIdx.x & (kWave - 1);
        if ((l & (kWave / VJ - 1)) == 0) red[half][a][(int)threadIdx.x / kWave + kWaves / VJ * (l / (kWave / VJ))] = s;
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < NV; a++) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < kWaves; q++) s += red[half][a][q];
        out[a] = s;
    }
    half ^= 1;
}

}  // namespace mp
