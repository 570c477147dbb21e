// Per-replica energy reduction (Eq. 1) for callers that cannot allocate
// device memory: spins and fields come from the caller's device buffers in
// natural site order, the energies go to a caller's device buffer, and the
// per-block partials live in a fixed device array of this file.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "rfim.h"
#include "rfim_internal.h"

namespace {

// (B, F) partial pairs; every GPU the library runs on holds its own copy
// until the process ends.
constexpr int kScratchPairs = RFIM_NOALLOC_MAX_PARTIALS;
constexpr int kMaxBlocks = 1024;        // partials per replica at most
constexpr int kThreads = 256;
constexpr int kMinBlocks = 4096;        // workgroups of a large call: two rounds of 8 per CU
constexpr int kMaxDevices = 64;

static __device__ __align__(256) double scratch[2 * kScratchPairs];

// v of the lane that the DPP control names, 0 where there is none or the row
// is masked.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or_zero(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, true);
    return __hiloint2double(hi, lo);
}

// Sum over the wave, in lane 63: rows of 16 lanes by shifts of 1, 2, 4 and 8,
// then row to row.  In registers; a butterfly of shuffles goes through the
// LDS once per step (20.4 us a call at L = 64, R = 192 with it, 19.6 so).
__device__ __forceinline__ double wave_total(double v) {
    v += dpp_or_zero<0x111, 0xF>(v);
    v += dpp_or_zero<0x112, 0xF>(v);
    v += dpp_or_zero<0x114, 0xF>(v);
    v += dpp_or_zero<0x118, 0xF>(v);
    v += dpp_or_zero<0x142, 0xA>(v);
    v += dpp_or_zero<0x143, 0xC>(v);
    return v;
}

// V consecutive spins as W dwords (V = 16 or 4), or one spin.
template <int V> struct Spins {
    static constexpr int W = V == 16 ? 4 : 1;
    int32_t w[W];
};

template <int V>
__device__ __forceinline__ Spins<V> load_spins(const int8_t *p) {
    Spins<V> v;
    if constexpr (V == 16) {
        const int4 q = *(const int4 *)p;
        v.w[0] = q.x;
        v.w[1] = q.y;
        v.w[2] = q.z;
        v.w[3] = q.w;
    } else if constexpr (V == 4) {
        v.w[0] = *(const int32_t *)p;
    } else {
        v.w[0] = *p;
    }
    return v;
}

// sum of s_q t_q over the V spins, added to acc (four int8 products per
// instruction)
template <int V>
__device__ __forceinline__ int dot_spins(const Spins<V> &s, const Spins<V> &t, int acc) {
    if constexpr (V == 1) {
        return acc + s.w[0] * t.w[0];
    } else {
#pragma unroll
        for (int w = 0; w < Spins<V>::W; ++w) acc = __builtin_amdgcn_sdot4(s.w[w], t.w[w], acc, false);
        return acc;
    }
}

// The workgroup's sums of RB replicas: the partials of block b or, if it is
// the only one, the energies.
template <int RB>
__device__ __forceinline__ void write_sums(const int (&bsum)[RB], const double (&fsum)[RB], int R, int nb, int b, int r0,
                                           double J, double h, double *part, double *E) {
    __shared__ double red[2 * RB][4];
    const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < RB; ++q) {
        const double wb = (double)__ockl_wfred_add_i32(bsum[q]), wf = wave_total(fsum[q]);
        if (lane == 63) {
            red[2 * q][wave] = wb;
            red[2 * q + 1][wave] = wf;
        }
    }
    __syncthreads();
    const int q = (int)threadIdx.x;
    if (q >= RB || r0 + q >= R) return;
    const double B = ((red[2 * q][0] + red[2 * q][1]) + red[2 * q][2]) + red[2 * q][3];
    const double F = ((red[2 * q + 1][0] + red[2 * q + 1][1]) + red[2 * q + 1][2]) + red[2 * q + 1][3];
    if (nb == 1) {
        E[r0 + q] = -(J * B) - (h * F);
    } else {
        double *o = part + 2 * ((size_t)(r0 + q) * nb + b);
        o[0] = B;
        o[1] = F;
    }
}

// Block (b, group g): sites [b * chunk, min(N, (b + 1) * chunk)) of replicas
// g * RB .. g * RB + RB - 1 (chunk a multiple of V).  B counts each bond once
// through its forward partner along x, y and z (periodic); F = sum f_i s_i in
// FP64.  A thread takes V consecutive sites of a row at a time (V divides L)
// and steps kThreads * V sites through the chunk, its coordinates carried
// along without divisions; the field of those sites is read and converted
// once for the RB replicas.  Per thread in site order, then over the wave
// (wave_total), then the four waves in order: the same sum on every call.
// nb = 1 writes the energies themselves.
//
// Bound: load latency and the L1 (each spin row is read for its own sites and
// as the forward row of two others); the spins are read from memory about
// once.  It takes the sizes whose rows are not whole 16-site units and arrays
// without their alignment: 32 us at L = 100, R = 50 (50 MB of spins).
template <int V, int RB>
__global__ __launch_bounds__(kThreads) void site_energy_partials(int L, int R, int nb, int N, int chunk, double J,
                                                                 double h, const int8_t *__restrict__ spins,
                                                                 const float *__restrict__ fields,
                                                                 double *__restrict__ part, double *__restrict__ E,
                                                                 int remap) {
    uint32_t blk = blockIdx.x;
    // blocks go round-robin to the 8 XCDs: a contiguous range each keeps the
    // forward planes in the same L2
    if (remap) blk = (blk & 7u) * (gridDim.x >> 3) + (blk >> 3);
    const int b = (int)(blk % (uint32_t)nb), r0 = (int)(blk / (uint32_t)nb) * RB;
    const int i0 = b * chunk, i1 = min(N, i0 + chunk);
    const int LL = L * L;
    // coordinates of this thread's first unit, and of a step of kThreads units
    int i = i0 + (int)threadIdx.x * V;
    int x = i % L, y = (i / L) % L, z = i / LL;
    const int step = kThreads * V, sx = step % L, sy = (step / L) % L, sz = step / LL;
    int bsum[RB];
    double fsum[RB];
    const int8_t *sp[RB];
#pragma unroll
    for (int q = 0; q < RB; ++q) {
        bsum[q] = 0;
        fsum[q] = 0.0;
        sp[q] = spins + (size_t)min(r0 + q, R - 1) * (size_t)N;   // past the last: read again, not written
    }
    for (; i < i1; i += step) {
        const int ix = x + V == L ? i + V - L : i + V;
        const int iy = y + 1 == L ? i - (L - 1) * L : i + L;
        const int iz = z + 1 == L ? i - (L - 1) * LL : i + LL;
        double f[V];
        if constexpr (V >= 4) {
#pragma unroll
            for (int q = 0; q < V; q += 4) {
                const float4 v = *(const float4 *)(fields + i + q);
                f[q] = v.x;
                f[q + 1] = v.y;
                f[q + 2] = v.z;
                f[q + 3] = v.w;
            }
        } else {
            f[0] = fields[i];
        }
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            const Spins<V> s = load_spins<V>(sp[q] + i);
            const Spins<V> sy1 = load_spins<V>(sp[q] + iy), sz1 = load_spins<V>(sp[q] + iz);
            Spins<V> sx1;
            if constexpr (V == 1) {
                sx1.w[0] = sp[q][ix];
            } else {
                // the V sites one further along the row
                const int32_t next = *(const uint8_t *)(sp[q] + ix);
#pragma unroll
                for (int w = 0; w < Spins<V>::W; ++w) {
                    const uint32_t hi = w + 1 < Spins<V>::W ? (uint32_t)s.w[w + 1 < Spins<V>::W ? w + 1 : 0] : (uint32_t)next;
                    sx1.w[w] = (int32_t)__builtin_amdgcn_alignbyte(hi, (uint32_t)s.w[w], 1u);
                }
            }
            bsum[q] = dot_spins<V>(s, sx1, dot_spins<V>(s, sy1, dot_spins<V>(s, sz1, bsum[q])));
#pragma unroll
            for (int k = 0; k < V; ++k) {
                const int si = V == 1 ? s.w[0] : (int)(int8_t)(s.w[k >> 2] >> (8 * (k & 3)));
                fsum[q] = fma(f[k], (double)si, fsum[q]);   // the product is exact
            }
        }
        x += sx;
        y += sy;
        z += sz;
        if (x >= L) {
            x -= L;
            ++y;
        }
        if (y >= L) {
            y -= L;
            ++z;
        }
    }
    write_sums<RB>(bsum, fsum, R, nb, b, r0, J, h, part, E);
}

// Rows of whole 16-site units (L a multiple of 16): a thread keeps one unit of
// the plane and walks `cz` planes up, so that the unit above is the next
// step's own; the sums as in site_energy_partials.  Block b of a group takes
// threads [256 b, 256 b + 256) of the (L / cz rounded up) * L * L / 16 columns.
// SHUF (L a power of two): a wave holds whole rows and the spin past a unit's
// end comes from the lane that has it; else it is a load of one byte.
//
// Bound: the FP64 field sum (three instructions per site) and the loads, by
// turns; the spins are read from memory once, their row ahead in y a second
// time from the L1.  L = 64, R = 192 (50 MB of spins): 16.5 us a call with the
// totals, 20.8 with each unit's three rows loaded for itself (136 with one site
// per thread step and 64-bit divisions); L = 128, R = 64 36 against 62.  The
// next plane's loads ahead of this one's sums: 18.6 and 38 (registers).
template <int RB, bool SHUF>
__global__ __launch_bounds__(kThreads) void site_energy_columns(int L, int R, int nb, int N, int cz, double J, double h,
                                                                const int8_t *__restrict__ spins,
                                                                const float *__restrict__ fields,
                                                                double *__restrict__ part, double *__restrict__ E,
                                                                int remap) {
    uint32_t blk = blockIdx.x;
    if (remap) blk = (blk & 7u) * (gridDim.x >> 3) + (blk >> 3);
    const int b = (int)(blk % (uint32_t)nb), r0 = (int)(blk / (uint32_t)nb) * RB;
    const int LL = L * L, rowu = L >> 4, upp = rowu * L;
    const int g = b * kThreads + (int)threadIdx.x, zc = g / upp, p = g - zc * upp;
    const int y = p / rowu, x = p - y * rowu;
    int z = zc * cz;
    const int z1 = min(z + cz, L);
    int i = z * LL + 16 * p;
    const int dx = x + 1 == rowu ? 16 - L : 16, dy = y + 1 == L ? -(L - 1) * L : L;
    const int next_lane = 4 * (int)(((threadIdx.x & 63u) - (uint32_t)x) + (x + 1 == rowu ? 0u : (uint32_t)x + 1u));
    int bsum[RB];
    double fsum[RB];
    const int8_t *sp[RB];
    Spins<16> s[RB];
#pragma unroll
    for (int q = 0; q < RB; ++q) {
        bsum[q] = 0;
        fsum[q] = 0.0;
        sp[q] = spins + (size_t)min(r0 + q, R - 1) * (size_t)N;   // past the last: read again, not written
        if (z < L) s[q] = load_spins<16>(sp[q] + i);
    }
    for (; z < z1; ++z) {
        const int iz = z + 1 == L ? i - (L - 1) * LL : i + LL;
        Spins<16> up[RB], sy[RB];
        int32_t next[RB];
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            up[q] = load_spins<16>(sp[q] + iz);
            sy[q] = load_spins<16>(sp[q] + i + dy);
            if (!SHUF) next[q] = *(const uint8_t *)(sp[q] + i + dx);
        }
        float4 f[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) f[k] = *(const float4 *)(fields + i + 4 * k);
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            if (SHUF) next[q] = __builtin_amdgcn_ds_bpermute(next_lane, s[q].w[0]);
            Spins<16> sx;
#pragma unroll
            for (int w = 0; w < 4; ++w)
                sx.w[w] = (int32_t)__builtin_amdgcn_alignbyte((uint32_t)(w < 3 ? s[q].w[w < 3 ? w + 1 : 0] : next[q]),
                                                              (uint32_t)s[q].w[w], 1u);
            bsum[q] = dot_spins<16>(s[q], sx, dot_spins<16>(s[q], sy[q], dot_spins<16>(s[q], up[q], bsum[q])));
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double fk[4] = {f[k].x, f[k].y, f[k].z, f[k].w};
#pragma unroll
            for (int q = 0; q < RB; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    fsum[q] = fma(fk[j], (double)(int)(int8_t)(s[q].w[k] >> (8 * j)), fsum[q]);   // the product is exact
        }
#pragma unroll
        for (int q = 0; q < RB; ++q) s[q] = up[q];
        i += LL;
    }
    write_sums<RB>(bsum, fsum, R, nb, b, r0, J, h, part, E);
}

// E_r = -(J B_r) - (h F_r): one wave per replica, lane l adds blocks l,
// l + 64, ... in order, then over the wave (wave_total).  (One thread per replica
// waited for its nb loads one after another.)
__global__ __launch_bounds__(kThreads) void site_energy_totals(int R, int nb, double J, double h,
                                                               const double *__restrict__ part,
                                                               double *__restrict__ E) {
    const int r = (int)(blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6)), lane = (int)threadIdx.x & 63;
    if (r >= R) return;
    const double2 *p = (const double2 *)part + (size_t)r * nb;
    double B = 0.0, F = 0.0;
    for (int b = lane; b < nb; b += 64) {
        const double2 v = p[b];
        B += v.x;
        F += v.y;
    }
    B = wave_total(B);
    F = wave_total(F);
    if (lane == 63) E[r] = -(J * B) - (h * F);
}

// The blocks of a call: nb per group of RB replicas.
struct Split {
    int nb, chunk;
};

// Enough workgroups to fill the chip, but at least one step of every thread
// in each, and no more partials than the scratch array and the totals take.
Split split_sites(int N, int V, int groups, int R) {
    const int unit = kThreads * V, units = (N + unit - 1) / unit;
    int nb = std::min(units, (kMinBlocks + groups - 1) / groups);
    nb = std::min(nb, std::min(kMaxBlocks, kScratchPairs / R));   // >= 1 since R <= kScratchPairs
    const int per = (units + nb - 1) / nb;                        // whole steps: no idle threads inside one
    return {(units + per - 1) / per, per * unit};
}

hipError_t launch_totals(int R, int nb, double J, double h, const double *part, double *E, hipStream_t s) {
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && nb > 1) {
        hipLaunchKernelGGL(site_energy_totals, dim3((unsigned)((R + 3) / 4)), dim3(kThreads), 0, s, R, nb, J, h, part, E);
        e = hipGetLastError();
    }
    return e;
}

template <int V, int RB>
hipError_t launch_energies(int L, int R, double J, double h, const int8_t *spins, const float *fields, double *part,
                           double *E, hipStream_t s) {
    const int N = L * L * L, groups = (R + RB - 1) / RB;
    const Split sp = split_sites(N, V, groups, R);
    const unsigned blocks = (unsigned)sp.nb * (unsigned)groups;
    hipLaunchKernelGGL((site_energy_partials<V, RB>), dim3(blocks), dim3(kThreads), 0, s, L, R, sp.nb, N, sp.chunk, J,
                       h, spins, fields, part, E, blocks % 8u == 0 ? 1 : 0);
    return launch_totals(R, sp.nb, J, h, part, E, s);
}

// Planes a thread walks: as many as leave kMinColumnBlocks workgroups, each of
// them full, and no more partials than the scratch array and the totals take.
// Two to four workgroups per CU are best: L = 64, R = 192 16.5 us with 768,
// 19.5 with 384 or 1536; L = 128, R = 40 27.6 us with 640, 42 with 1280, 33
// with 320; R = 64 36 with 512, 45 with 1024.
constexpr int kMinColumnBlocks = 512;

template <int RB>
hipError_t launch_columns(int L, int R, double J, double h, const int8_t *spins, const float *fields, double *part, double *E,
                          hipStream_t s) {
    const int N = L * L * L, groups = (R + RB - 1) / RB, upp = L * L / 16;
    auto blocks_of = [&](int cz) { return (int)(((long long)((L + cz - 1) / cz) * upp + kThreads - 1) / kThreads); };
    const int most = std::min(kMaxBlocks, kScratchPairs / R);
    int cz = 1;
    while (cz < L && (blocks_of(cz) > most || ((long long)L * upp >= 2ll * cz * kThreads &&
                                               (long long)blocks_of(2 * cz) * groups >= kMinColumnBlocks)))
        cz *= 2;
    const int nb = blocks_of(cz);
    if (nb > most) return launch_energies<4, RB>(L, R, J, h, spins, fields, part, E, s);   // R beyond 10^5
    const unsigned blocks = (unsigned)nb * (unsigned)groups;
    if ((L & (L - 1)) == 0)
        hipLaunchKernelGGL((site_energy_columns<RB, true>), dim3(blocks), dim3(kThreads), 0, s, L, R, nb, N, cz, J, h, spins,
                           fields, part, E, blocks % 8u == 0 ? 1 : 0);
    else
        hipLaunchKernelGGL((site_energy_columns<RB, false>), dim3(blocks), dim3(kThreads), 0, s, L, R, nb, N, cz, J, h, spins,
                           fields, part, E, blocks % 8u == 0 ? 1 : 0);
    return launch_totals(R, nb, J, h, part, E, s);
}

std::mutex g_mu;
double *g_scratch[kMaxDevices] = {};

// The device address of this GPU's copy of `scratch`, looked up once per
// device with that device current.  In host code the array's name is not a
// device address; only this pointer may reach kernels.
int scratch_on_current_device(double **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return rfim_host::set_error(RFIM_EDEVICE, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return rfim_host::set_error(RFIM_EDEVICE, "device %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_mu);
    if (!g_scratch[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return rfim_host::set_error(RFIM_EDEVICE, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
        g_scratch[dev] = (double *)p;
    }
    *out = g_scratch[dev];
    return RFIM_OK;
}

}  // namespace

extern "C" int rfim_energies_noalloc(int L, int R, double J, double h, const int8_t *d_spins,
                                     const float *d_fields, double *d_E, void *hip_stream) {
    if (L < 2 || L > 1024 || (L & 1))
        return rfim_host::set_error(RFIM_EINVAL, "L must be even with 2 <= L <= 1024 (got %d)", L);
    if (R < 1) return rfim_host::set_error(RFIM_EINVAL, "R must be >= 1 (got %d)", R);
    if (R > kScratchPairs)
        return rfim_host::set_error(RFIM_ECAP, "R = %d beyond the %d replicas the fixed partial array holds", R,
                                    kScratchPairs);
    if (!d_spins || !d_fields || !d_E) return rfim_host::set_error(RFIM_EINVAL, "NULL device pointer");
    if (!std::isfinite(J) || !std::isfinite(h)) return rfim_host::set_error(RFIM_EINVAL, "J and h must be finite");
    double *part = nullptr;
    int rc = scratch_on_current_device(&part);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)hip_stream;
    // Widest step that divides a row, where both arrays allow its loads.  Two
    // replicas share a pass over the field (L = 64, R = 192: 16.5 us with two,
    // 21 with one, 18 with four).
    const bool a16 = ((uintptr_t)d_fields & 15u) == 0;
    hipError_t e;
    if (L % 16 == 0 && a16 && ((uintptr_t)d_spins & 15u) == 0)
        e = R >= 2 ? launch_columns<2>(L, R, J, h, d_spins, d_fields, part, d_E, s)
                   : launch_columns<1>(L, R, J, h, d_spins, d_fields, part, d_E, s);
    else if (L % 4 == 0 && a16 && ((uintptr_t)d_spins & 3u) == 0)
        e = R >= 2 ? launch_energies<4, 2>(L, R, J, h, d_spins, d_fields, part, d_E, s)
                   : launch_energies<4, 1>(L, R, J, h, d_spins, d_fields, part, d_E, s);
    else
        e = R >= 2 ? launch_energies<1, 2>(L, R, J, h, d_spins, d_fields, part, d_E, s)
                   : launch_energies<1, 1>(L, R, J, h, d_spins, d_fields, part, d_E, s);
    if (e != hipSuccess) return rfim_host::set_error(RFIM_EDEVICE, "energy launch: %s", hipGetErrorString(e));
    return RFIM_OK;
}
