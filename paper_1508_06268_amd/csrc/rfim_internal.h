// Internal interface between the host runtime (rfim_api.hip) and the
// device kernels (rfim_kernels.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rfim_dev {

// Device layout of one realization (all arrays in HBM):
//   spins  uint8 [R_cap][2][N/2]  colour-split; byte = 1 iff s = +1.
//          Colour c, sublattice index j holds site 2j or 2j+1 (whichever has
//          colour c).
//   fbits  uint8 [2][N/2]         +-1 fields: byte = 4 iff h_i = +1, else 0.
//   fhf    float [2][N/2]         continuous fields: (float)(h * h_i - 6 J).
//   fraw   float [2][N/2]         continuous fields: h_i as given.
//   thr    uint32 [R_cap][32]     per slot, +-1 fields, indexed by
//                                 (up << 2) | (b << 1) | f with up = number of
//                                 +1 neighbours, b = spin byte, f = field bit:
//                                 a flip is taken iff u32 <= entry, unless bit
//                                 idx of entry 31 (the slot's never mask) is
//                                 set.  Entry = 0xFFFFFFFF where dE <= 0,
//                                 else floor(e^(-beta dE) 2^32) - 1, or 0 with
//                                 the never bit where that floor is 0.
//   betaf  float [R_cap]          per slot, continuous fields.
//   beta   double [R_cap]         per slot (exchange).
//   t2r, r2t int32 [R_cap]; att, acc uint64 [R_cap]
//   ctrs   uint64 [2]             global sweep counter t, exchange counter k.
//   part   double [nblk][R_cap][3] energy partials (B, F, M) per block,
//                                 block-major so that consecutive replicas'
//                                 partials of one block are adjacent (the
//                                 reduction reads them coalesced);
//                                 nblk = blocks_per_replica(shape).
//   E      double [R_cap]         energy by replica id after a reduction.
//   Mr     double [R_cap]         magnetisation by replica id (same reduction).
//   obs    double [R_cap][6]      per slot, one sample per exchange step
//                                 (Sec. 7): count, sum E, sum E^2, sum |M|,
//                                 sum M^2, sum M^4.
struct Lattice {
    int L, N, half, R;          // R = replicas currently active
    int log2L;                  // >= 3 when L is a power of two, else -1
    int kind;                   // 0 bimodal, 1 continuous
    float Jf;
    double J, h;
    uint32_t key0, key1, rho;
    uint8_t *spins;
    const uint8_t *fbits;
    const float *fhf, *fraw;
    const uint32_t *thr;
    const float *betaf;
    const double *beta;
    int32_t *t2r, *r2t;
    uint64_t *att, *acc;
    uint64_t *ctrs;
    double *part;
    int nblk;                   // energy partials per replica
    int pstride;                // replicas per block row of part (R_cap)
    int mode;                   // power-of-two L: 0 streaming, 1 LDS-resident
    int nw, wg;                 // dwords per thread, threads per workgroup
    double *E;
    double *Mr;
    double *obs;
    // one bit per spin (rfim_set_spin_storage): bits uint32 [R_cap][2][N/64],
    // colour c, word w = sublattice indices 32w..32w+31 (index 32w+4b+q at
    // bit 8q+b), 1 iff s = +1; fbw uint32 [2][N/64] in the same order,
    // 1 iff h_i = +1 (+-1 fields).  Null while the spins live in `spins`.
    // fhw float [2][N/2]: continuous fields as in fhf, ordered for the bit
    // sweep: in colour c, the four values of sublattice indices
    // 32w+4b..32w+4b+3 (block b of word w) are float4 number
    // (8 (w/64) + b) 64 + w%64, so that the 64 threads of a wavefront read
    // block b of their words as 1 KiB in one piece (N/64 is a multiple of
    // 64 at every L that bit storage takes).
    uint32_t *bits;
    const uint32_t *fbw;
    const float *fhw;
    // Fourier measurement (null while it is off): fpart int32
    // [R_cap][L][2L] scratch, trig double [2][L] = cos, sin of 2 pi v / L,
    // fobs double [R_cap][2] = (count, sum F) by slot.
    int32_t *fpart;
    const double *trig;
    double *fobs;
};

// Above this many workgroups per replica the streaming sweep does not write
// energy partials; a separate energy kernel with 64 blocks does.
constexpr int kMaxFusedBlocks = 1024;

// Launch shapes.  Power-of-two L >= 8: mode 0 (streaming: one chunk of
// nw dwords per thread, wg in {64, 128, 256}), mode 1 (LDS-resident,
// L <= 32: one workgroup of wg threads per replica runs every sweep of an
// exchange interval) or modes 2..4 (slabs, L = 16..64: nw slabs per
// replica, mode - 1 sweeps per launch, wg threads).  Other L: generic
// kernel, shape (0, 0, 0).  Every shape gives bit-identical results.
bool shape_valid(int L, int mode, int nw, int wg);
// Batch and pool classes also take shape (kModeBits, 0, 0) at L = 64, 128
// or 256: one bit per spin, each item swept on its own by the bit sweep
// (the storage of a standalone handle is set with rfim_set_spin_storage
// instead).
constexpr int kModeBits = 5;
// Energy partials per replica for a shape (1 for resident, the workgroups
// per replica when the streaming sweep fuses the energy, else 64).
int blocks_per_replica(int L, int mode, int nw, int wg);
// Workgroups per replica of one streaming half-sweep launch.
int stream_blocks_per_replica(int L, int nw, int wg);
// True when the sweep kernels themselves write the energy partials.
bool fused_energy(const Lattice &lat);

// One realization's interval kernels (resident, slab, box) can take the
// exchange step before their first sweep: every workgroup decides the pair of
// its own replica from the partials of the previous interval, so that an
// interval is its sweep launches alone.  The step reads one copy of the
// permutation and of the partials and writes the other (a workgroup that ends
// early must not change what one that starts late still reads); the counters
// come from the host.  r2t null: no such step, everything from the descriptor.
struct StepIn {
    const int32_t *r2t = nullptr, *t2r = nullptr;   // the permutation to sweep by, or before the step
    const double *part = nullptr;                   // null: no step is pending
    int32_t *r2t_out = nullptr, *t2r_out = nullptr; // the permutation after it
    double *part_out = nullptr;                     // where this interval's partials go
    uint64_t k = 0;                                 // the step's exchange counter
    uint32_t t0 = 0;                                // the sweep counter
    int nblk = 1, per = 1;                          // the order the partials are added in (partials_per_range)
};
// The totals of nblk partials of R replicas are added in ranges of this many,
// each in order, then the ranges in order.
int partials_per_range(int R, int nblk);
// Most replicas whose exchange step runs in one pass of a workgroup, and most
// partials per replica a step before the sweeps adds.
constexpr int kExchangeThreads = 1024, kMaxStepPartials = 8;

// One launch over a set of realizations that share L, field kind and shape:
// lats = device array of descriptors; map = one entry per workgroup:
// x = (realization << 16) | replica, y = block within the replica
// (streaming) or 0 (resident).
struct Launch {
    const Lattice *lats;
    const uint2 *map;
    int nblocks;
    int L, kind, mode, nw, wg;
    // one realization: its descriptor, passed by value (lats and map
    // unused; blocks enumerate (replica, block) in order, from replica r0)
    const Lattice *single = nullptr;
    int r0 = 0;
};

// Slab sweeps (mode 2..4, L = 16 or 32): nslab workgroups per replica, each
// a z-slab of L/nslab planes with the halo recomputed, mode - 1 sweeps per
// launch at most; reads `src`, writes `dst` (a second spin buffer: the
// workgroups of a replica must not see each other's new planes).
int slab_sweeps_per_launch(int mode);
size_t slab_lds_bytes(int L, int mode, int nslab);
int slab_positions_per_thread(int L, int mode, int nslab, int wg);
hipError_t launch_slab_sweep(const Lattice &lat, const StepIn &in, const uint8_t *src, uint8_t *dst, int mode, int nslab,
                             int wg, int nsweep, int toff, int energy, hipStream_t s);

// Double-checkerboard order with multi-hit updates (Sec. 3.2, Sec. 5.2):
// tiles of tx * ty * tz sites, `hits` local sweeps per tile visit.  Valid
// for L = 2^l >= 16 with tx a multiple of 8, every side dividing L into an
// even number of tiles, (tx / 8) ty tz threads per workgroup in
// {64, 128, ..., 1024}, the staged box within 64 KB of LDS, 1 <= hits <=
// 65536.
struct TileShape {
    int tx, ty, tz, hits;
};
bool tile_shape_valid(int L, const TileShape &ts);
size_t tile_lds_bytes(const TileShape &ts);
// The tiles of coarse colour `coarse` of every replica at sweep t + toff.
hipError_t launch_tile_sweep(const Lattice &lat, const TileShape &ts, int coarse, int toff, hipStream_t s);

// One bit per spin: L = 2^l with 64 <= L <= 256.  Workgroups per replica
// of a bit half-sweep (each writes one energy partial with ENERGY).
bool bits_valid(int L);
int bits_blocks_per_replica(int L);
// Half-sweep of colour `colour` at sweep t + toff for replicas r0..r0+nrep-1
// (energy != 0 on colour 1: also the energy partials of the final state).
hipError_t launch_bits_sweep(const Lattice &lat, int r0, int nrep, int colour, int toff, int energy, hipStream_t s);
// The bit sweep over a batch class in bit storage: ln.map holds one entry
// per replica (x = (realization << 16) | replica), ln.nblocks entries.
hipError_t launch_bits_batch(const Launch &ln, int colour, int toff, int energy, hipStream_t s);
// Byte spins <-> bit spins of replicas [0, R) (and, to bits, the +-1 field
// words).
hipError_t launch_pack_bits(const Lattice &lat, hipStream_t s);
hipError_t launch_unpack_bits(const Lattice &lat, hipStream_t s);

hipError_t launch_init(const Lattice &lat, int r0, int r1, hipStream_t s);
// Streaming half-sweep of colour `colour` at sweep t + toff (power-of-two
// L); energy != 0 on colour 1 also writes the energy partials.
hipError_t launch_stream_sweep(const Launch &ln, int colour, int toff, int energy, hipStream_t s);
// Resident: nsweep whole sweeps in one launch (energy != 0: also the
// energy partials of the final state).
hipError_t launch_resident(const Launch &ln, const StepIn &in, int nsweep, int energy, hipStream_t s);
// Other even L, one realization: half-sweeps (any L), or whole sweeps of
// LDS-resident replicas with the energy partials of the final state: for L = 4
// and the small L whose planes do not split into whole Philox blocks (L % 4 ==
// 2; the others have boxes, below), as long as one workgroup sweeps a replica
// in less time than two launches take (us a sweep at R = 32, resident against
// half-sweeps: 2.8 and 7.8 at L = 10; about even at L = 26).
constexpr int kGenericResidentMaxL = 22;
bool generic_resident(int L);
hipError_t launch_generic_resident(const Lattice &lat, const StepIn &in, int nsweep, int energy, hipStream_t s);
// Boxes (L a multiple of 4, not a power of two): slabs of `planes` planes, up
// to `sweeps` whole sweeps a launch, from src to dst (a second spin buffer).
// box_plan: the split for R replicas, planes = 0 where half-sweeps or the
// resident form are the better one.
constexpr int kMaxBoxSlabs = 64;            // one energy partial each
constexpr int kBoxMaxL = 88;                // a plane's blocks within one workgroup's threads
struct BoxPlan {
    int planes, sweeps;
};
BoxPlan box_plan(int L, int R);
hipError_t launch_box(const Lattice &lat, const StepIn &in, const uint8_t *src, uint8_t *dst, const BoxPlan &plan,
                      int nsweep, int toff, int energy, hipStream_t s);
hipError_t launch_generic_sweep(const Lattice &lat, int colour, int toff, hipStream_t s);
// Energy partials of the state at rest, lat.nblk per replica, from the bytes
// or, in bit storage, the bits.
hipError_t launch_energy(const Lattice &lat, hipStream_t s);
// Energies and magnetisations to the arrays that are not null (pinned host
// memory): by replica id, E_slot and M_slot by temperature slot.  Each
// workgroup that writes any sets its word of `done` (pinned, cleared by the
// caller) to 1 after its writes: readout_flags words, copy_out_flags for
// CopyOut.
struct Readout {
    int64_t *B = nullptr;
    double *F = nullptr;
    int64_t *M = nullptr;
    double *E_slot = nullptr;
    int64_t *M_slot = nullptr;
    uint32_t *done = nullptr;
};
unsigned readout_flags(const Lattice &lat);
hipError_t launch_readout(const Lattice &lat, const Readout &out, hipStream_t s);
// Up to kMax device arrays of whole dwords to pinned host memory.
struct CopyOut {
    static constexpr int kMax = 3;
    const void *src[kMax] = {};
    void *dst[kMax] = {};
    uint32_t words[kMax] = {};
    uint32_t *done = nullptr;
};
unsigned copy_out_flags(const CopyOut &c);
// Zeros to two arrays of 8-byte words (either may be empty).
hipError_t launch_clear(void *a, size_t na, void *b, size_t nb, hipStream_t s);
hipError_t launch_copy_out(const CopyOut &c, hipStream_t s);
// Configurations (+-1, natural site order; sites first .. first + count - 1 of
// the replicas' [R][N], both multiples of 64 or of a replica) to and from
// pinned host memory, in either storage, and the fields of a realization from
// it (first and count multiples of 4).
hipError_t launch_spins_out(const Lattice &lat, size_t first, size_t count, int8_t *dst, hipStream_t s);
hipError_t launch_spins_in(const Lattice &lat, size_t first, size_t count, const int8_t *src, hipStream_t s);
hipError_t launch_fields_in(const Lattice &lat, size_t first, size_t count, const float *src, hipStream_t s);
// One exchange step for each of the n realizations in lats (device array);
// with `in` (n = 1) the step pending there, which brings the permutation, the
// counters (tadv sweeps, step in.k) and the rest back to the descriptor.
hipError_t launch_exchange(const Lattice *lats, int n, int tadv, const StepIn &in, hipStream_t s);
hipError_t launch_advance(const Lattice &lat, int tadv, hipStream_t s);
// Fourier observable of every replica, accumulated by slot (rfim_measure.hip),
// through the descriptor's fpart, trig and fobs.
hipError_t launch_fourier(const Lattice &lat, hipStream_t s);
// The same for the measured items of a batch: map entries x = (realization <<
// 16) | replica with, in `chunks`, y = (planes per chunk << 16) | chunk
// (fourier_chunk_planes(L) planes each) and, in `replicas` (those of more than
// one chunk), y = the number of chunks.  L a power of two in [8, max_l].
int fourier_chunk_planes(int L);
hipError_t launch_fourier_batch(const Lattice *lats, const uint2 *chunks, int nchunks, const uint2 *replicas, int nreplicas,
                                int max_l, hipStream_t s);

}  // namespace rfim_dev

namespace rfim_host {
// Records a message for rfim_last_error() (printf-style) and returns code.
int set_error(int code, const char *fmt, ...);
}  // namespace rfim_host
