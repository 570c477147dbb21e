// Fourier observable of the correlation length (arXiv:1508.06268, Sec. 7)
// on the device, one sample per exchange step and temperature slot:
//   F = (1/(3N)) sum_mu [(sum_i s_i cos(K x_mu,i))^2 + (sum_i s_i sin(K x_mu,i))^2],
// K = 2 pi / L, mu over the three axes (the printed sums carry the field
// h_i; read with the spins s_i, the usual second-moment estimator).  Each
// inner sum is grouped by coordinate: integer plane sums n_mu(v) first
// (exact in any order), then sum_v cos(K v) n_mu(v) in FP64 with v
// ascending, so the result does not depend on the launch shape.
//
// Compiled with -ffp-contract=off like the other kernels.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "rfim_internal.h"

namespace rfim_dev {

namespace {

// Descriptor pointers are generic; typed as global they are read by global_*
// instructions, which the compiler may move past LDS accesses.
#define GAS __attribute__((address_space(1)))

// A replica is taken in chunks of whole z-planes, one workgroup each: all of
// it up to this many sites (the workgroup then goes on to F), else about half
// of that.
constexpr int kWholeSites = 32768;

int chunk_planes(int L) {
    if ((long long)L * L * L <= kWholeSites) return L;
    return std::max(2, std::min(L, kWholeSites / 2 / (L * L)));
}

// C_mu, S_mu and F in FP64 from the plane sums n[mu][v] (in LDS), added to
// the replica's current slot: lane 2 mu + q of the first wave takes one of
// the six sums over v, ascending, lane 0 puts F together.
__device__ __forceinline__ void add_sample(const Lattice &lat, uint32_t r, const int32_t (*n)[1024]) {
    extern __shared__ double trig[];                    // [2][L]; the caller's barrier covers it
    if (threadIdx.x >= 64u) return;
    const int L = lat.L, lane = (int)threadIdx.x;
    double acc = 0.0;
    if (lane < 6) {
        const double *t = trig + (lane & 1 ? L : 0);
        const int32_t *nv = n[lane >> 1];
#pragma unroll 8
        for (int v = 0; v < L; ++v) acc += t[v] * (double)nv[v];
    }
    const double c0 = __shfl(acc, 0, 64), s0 = __shfl(acc, 1, 64), c1 = __shfl(acc, 2, 64), s1 = __shfl(acc, 3, 64),
                 c2 = __shfl(acc, 4, 64), s2 = __shfl(acc, 5, 64);
    if (lane != 0) return;
    const double F = (c0 * c0 + s0 * s0 + c1 * c1 + s1 * s1 + c2 * c2 + s2 * s2) / (3.0 * (double)lat.N);
    double *o = lat.fobs + 2 * (size_t)lat.r2t[r];
    o[0] += 1.0;
    o[1] += F;
}

// The cosines and sines into LDS, where the chain of FP64 additions reads
// them.
__device__ __forceinline__ void stage_trig(const Lattice &lat) {
    extern __shared__ double trig[];
    for (int v = (int)threadIdx.x; v < 2 * lat.L; v += 256) trig[v] = ((GAS const double *)lat.trig)[v];
}

// Plane sums of chunk `ch` of replica r (up spins along x, y and z, then
// 2 up - sites): to the partials, or, when the chunk is the whole replica, on
// to F.  ROWS (L a multiple of 8): a thread keeps a dword column w of the row
// and takes every few rows; in row (y, z) colour (y + z) mod 2 holds the even
// x.  The column sums stay in registers as packed bytes (at most 255 rows
// between two flushes), row sums are one byte sum and one LDS addition.
//
// Bound: memory latency and the launches.  The Binder study's 43 realizations
// (15 replicas each) took two launches per realization and step, each plane a
// wave's walk over its rows byte by byte: 860 launches of 4 to 21 us a run of
// 10 steps, now 20 of 14.5 and 4.4 us.
template <bool ROWS, bool BATCH>
__global__ __launch_bounds__(256) void fourier_sums(Lattice lat0, const Lattice *__restrict__ lats,
                                                    const uint2 *__restrict__ map, int nchunk, int planes) {
    __shared__ int32_t n[3][1024];
    uint32_t r, ch;
    if (BATCH) {
        const uint2 e = map[blockIdx.x];
        r = e.x & 0xFFFFu;
        ch = e.y & 0xFFFFu;
        planes = (int)(e.y >> 16);
    } else {
        r = blockIdx.x / (uint32_t)nchunk;
        ch = blockIdx.x % (uint32_t)nchunk;
    }
    const Lattice &lat = BATCH ? lats[map[blockIdx.x].x >> 16] : lat0;
    const uint32_t L = (uint32_t)lat.L, Lh = L >> 1, half = (uint32_t)lat.half;
    const uint32_t z0 = ch * (uint32_t)planes, nz = min((uint32_t)planes, L - z0);
    for (uint32_t v = threadIdx.x; v < L; v += 256u) n[0][v] = n[1][v] = n[2][v] = 0;
    if (nz == L) stage_trig(lat);
    __syncthreads();
    GAS const uint8_t *s0 = (GAS const uint8_t *)lat.spins + (size_t)r * lat.N, *s1 = s0 + half;
    if (ROWS) {
        const uint32_t wpr = Lh >> 2, per = 256u / wpr;               // dwords of a row, rows at a time
        const uint32_t w = threadIdx.x % wpr, first = threadIdx.x / wpr;
        if (first < per) {
            constexpr uint32_t B = 8;                                   // rows whose loads go out together
            const uint32_t end = nz * L, dy = per % L, dz = per / L;
            uint32_t even = 0, odd = 0, rows = 0, y = first % L, z = z0 + first / L;
            int plane_up = 0;
            for (uint32_t q0 = first; q0 < end; q0 += B * per) {
                uint32_t a[B], b[B];
#pragma unroll
                for (uint32_t k = 0; k < B; ++k) {
                    const uint32_t q = min(q0 + k * per, end - 1u);     // past the end: read again, not used
                    const uint32_t j = (z0 * L + q) * Lh + 4u * w;
                    a[k] = *(GAS const uint32_t *)(s0 + j);
                    b[k] = *(GAS const uint32_t *)(s1 + j);
                }
#pragma unroll
                for (uint32_t k = 0; k < B; ++k) {
                    const uint32_t q = q0 + k * per;
                    if (q >= end) break;
                    const bool swap = ((y + z) & 1u) != 0;              // colour 1 holds the even x
                    even += swap ? b[k] : a[k];
                    odd += swap ? a[k] : b[k];
                    const int up = (int)__builtin_amdgcn_sad_u8(a[k], 0u, __builtin_amdgcn_sad_u8(b[k], 0u, 0u));
                    atomicAdd(&n[1][y], up);
                    plane_up += up;
                    const uint32_t zq = z;
                    z += dz;
                    y += dy;
                    if (y >= L) {
                        y -= L;
                        ++z;
                    }
                    if (z != zq || q + per >= end) {
                        atomicAdd(&n[2][zq], plane_up);
                        plane_up = 0;
                    }
                    if (++rows == 255u || q + per >= end) {
                        rows = 0;
#pragma unroll
                        for (uint32_t i = 0; i < 4; ++i) {
                            atomicAdd(&n[0][2u * (4u * w + i)], (int)((even >> (8u * i)) & 0xFFu));
                            atomicAdd(&n[0][2u * (4u * w + i) + 1u], (int)((odd >> (8u * i)) & 0xFFu));
                        }
                        even = odd = 0;
                    }
                }
            }
        }
    } else {
        for (uint32_t q = threadIdx.x; q < nz * L * Lh; q += 256u) {
            const uint32_t m = q % Lh, y = (q / Lh) % L, z = z0 + q / (Lh * L);
            const uint32_t j = (z * L + y) * Lh + m, a = s0[j], b = s1[j];
            const bool swap = ((y + z) & 1u) != 0;
            atomicAdd(&n[0][2u * m], (int)(swap ? b : a));
            atomicAdd(&n[0][2u * m + 1u], (int)(swap ? a : b));
            atomicAdd(&n[1][y], (int)(a + b));
            atomicAdd(&n[2][z], (int)(a + b));
        }
    }
    __syncthreads();
    const int32_t line = (int32_t)(L * nz);                             // sites behind n[0][v] and n[1][v]
    if (nz == L) {
        for (uint32_t v = threadIdx.x; v < L; v += 256u)
#pragma unroll
            for (int mu = 0; mu < 3; ++mu) n[mu][v] = 2 * n[mu][v] - line;
        __syncthreads();
        add_sample(lat, r, n);
        return;
    }
    // partials of a replica: [chunk][2L] (x, y), then its z-planes
    int32_t *part = lat.fpart + (size_t)r * L * 2u * L;
    for (uint32_t v = threadIdx.x; v < L; v += 256u) {
        part[(size_t)ch * 2u * L + v] = 2 * n[0][v] - line;
        part[(size_t)ch * 2u * L + L + v] = 2 * n[1][v] - line;
        if (v < nz) part[(size_t)((L + (uint32_t)planes - 1u) / (uint32_t)planes) * 2u * L + z0 + v] =
            2 * n[2][z0 + v] - (int32_t)(L * L);
    }
}

// F of a replica taken in several chunks.
template <bool BATCH>
__global__ __launch_bounds__(256) void fourier_samples(Lattice lat0, const Lattice *__restrict__ lats,
                                                       const uint2 *__restrict__ map, int nchunk) {
    __shared__ int32_t n[3][1024];
    if (BATCH) nchunk = (int)map[blockIdx.x].y;
    const Lattice &lat = BATCH ? lats[map[blockIdx.x].x >> 16] : lat0;
    const uint32_t r = BATCH ? (map[blockIdx.x].x & 0xFFFFu) : blockIdx.x, L = (uint32_t)lat.L;
    GAS const int32_t *part = (GAS const int32_t *)lat.fpart + (size_t)r * L * 2u * L;
    stage_trig(lat);
    for (uint32_t v = threadIdx.x; v < L; v += 256u) {
        int32_t nx = 0, ny = 0;
#pragma unroll 8
        for (int c = 0; c < nchunk; ++c) {
            nx += part[(size_t)c * 2u * L + v];
            ny += part[(size_t)c * 2u * L + L + v];
        }
        n[0][v] = nx;
        n[1][v] = ny;
        n[2][v] = part[(size_t)nchunk * 2u * L + v];
    }
    __syncthreads();
    add_sample(lat, r, n);
}

}  // namespace

int fourier_chunk_planes(int L) { return chunk_planes(L); }

hipError_t launch_fourier(const Lattice &lat, hipStream_t s) {
    const int planes = chunk_planes(lat.L), nchunk = (lat.L + planes - 1) / planes;
    const dim3 grid((unsigned)lat.R * (unsigned)nchunk);
    const size_t lds = 2 * (size_t)lat.L * sizeof(double);
    if (lat.L % 8 == 0)
        hipLaunchKernelGGL((fourier_sums<true, false>), grid, dim3(256), lds, s, lat, nullptr, nullptr, nchunk, planes);
    else
        hipLaunchKernelGGL((fourier_sums<false, false>), grid, dim3(256), lds, s, lat, nullptr, nullptr, nchunk, planes);
    if (nchunk > 1)
        hipLaunchKernelGGL((fourier_samples<false>), dim3((unsigned)lat.R), dim3(256), lds, s, lat, nullptr, nullptr, nchunk);
    return hipGetLastError();
}

hipError_t launch_fourier_batch(const Lattice *lats, const uint2 *chunks, int nchunks, const uint2 *replicas, int nreplicas,
                                int max_l, hipStream_t s) {
    const size_t lds = 2 * (size_t)max_l * sizeof(double);
    if (nchunks > 0)
        hipLaunchKernelGGL((fourier_sums<true, true>), dim3((unsigned)nchunks), dim3(256), lds, s, Lattice{}, lats, chunks, 1, 1);
    if (nreplicas > 0)
        hipLaunchKernelGGL((fourier_samples<true>), dim3((unsigned)nreplicas), dim3(256), lds, s, Lattice{}, lats, replicas, 1);
    return hipGetLastError();
}

}  // namespace rfim_dev
