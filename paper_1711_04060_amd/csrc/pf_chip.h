// pf_chip.h -- interface of the on-chip Krylov kernel (pf_chip.hip): a whole
// BiCGSTAB run of a grid whose vectors fit the registers and LDS of the chip,
// in one launch.
#pragma once

#include "pf_device.h"
#include <stddef.h>

namespace pfk {

constexpr int CH_NT = 512;      // threads per workgroup (tile)
constexpr int CH_LP = 616;      // LDS elements per staged plane; the last one takes masked stores
constexpr int CH_NQ = 5;        // sums per phase (at most)
constexpr int CH_GMAX = 256;    // tiles of one system (one per CU)
constexpr int CH_SPIN = 1 << 19;   // polls of one wait before a tile gives up

// bytes of the exchanged sums: two buffers of the tiles' and of the groups'
// (16-byte words), and the tiles' XCD ids
constexpr size_t CH_SUMS = 2 * CH_NQ * (CH_GMAX + 8) * 16 + CH_GMAX * 8;

// xy halo nodes kept per thread
constexpr int chip_halo_slots(int kz) { return kz <= 4 ? 1 : kz <= 8 ? 2 : 3; }

// boundary values published per thread
constexpr int chip_face_slots(int kz) { return kz <= 4 ? 3 : kz <= 8 ? 4 : 5; }

// operator forms: constant coefficient (PF1), palette coefficients without a
// shift, with a shift per node, with a shift per palette class
enum { CHF_CEPS = 0, CHF_NONE = 1, CHF_NODE = 2, CHF_CLASS = 3 };

// Partition of a grid's unknowns (Dirichlet faces left out) into c[0] x c[1]
// x c[2] tiles, sizes along each axis differing by at most one.
struct ChipGeom {
    int KZ = 0;                 // planes per tile the kernel instance holds (0: the grid does not fit)
    int o[3], n[3];             // first unknown and their count per axis
    int c[3];
    int G = 0;
    int fx = 0, fy = 0, fz = 0; // largest face of a tile normal to x, y, z, in whole cache lines
    int fstride = 0;            // exchange elements of a tile: 2 (fx + fy + fz)
};

// One system of a launch.
template <typename T>
struct ChipSys {
    int nx, ny, nz, P;
    ChipGeom ge;
    int zero_x;                 // start from x = 0 (x is not read)
    T ceps, cdiag, cidiag;      // CHF_CEPS
    uint8_t dirbit;
    const uint8_t *flags;       // CHF_CEPS: Dirichlet rows have bit dirbit
    const uint8_t *epsi;        // palette index per node, bit 7 = Dirichlet row
    const T *ftab, *stab;       // face table, shift per class (CHF_CLASS)
    const T *sig;               // CHF_NODE
    const T *s0;                // start vector r^ = D^-1 r
    const float *rt;            // shadow residual
    T *x;
    T *xtile;                   // KZ = 16: [G][KZ][CH_NT], x while the run lasts
    Scalars *sc;
    Scalars init;               // scalar block of the start
    void *face;                 // [2][G][fstride] exchanged boundary values (tagged: 2 sizeof(T) bytes each)
    void *sums;                 // exchanged partial sums and XCD ids (CH_SUMS bytes)
    unsigned tag0;              // tag of phase 0; phases count up from it
    int spin;                   // polls of one wait before a tile gives up
};

// Partition for a grid of nx x ny x nz nodes (Neumann faces: bit f of neu), at
// most gcap tiles and kzmax planes per tile; KZ = 0 when it does not fit.
ChipGeom chip_partition(int nx, int ny, int nz, int neu, int gcap, int kzmax);

// Device memory of a run by the instance of kz planes, in two blocks that
// never trade places: `tagged` bytes of {value, tag} words (the sums, and up to
// 8 planes the boundary values at `face`) whose readers take a word for an
// arrived one by its tag, and `plain` bytes of values without tags (16 planes:
// the boundary values at `face`, x of the tiles at `xtile`).
struct ChipSpace {
    size_t tagged, plain, face, xtile;
};
ChipSpace chip_space(const ChipGeom &ge, int kz, size_t elem);

// Dynamic LDS of a workgroup.
size_t chip_lds(int kz, size_t elem);

// Writes the scalar blocks and (one) stores the system into table[0].
template <typename T>
hipError_t chip_start(const ChipSys<T> *one, ChipSys<T> *table, int nsys, hipStream_t s);

// The Krylov runs of nsys systems of one form: tiles first[i] <= b < first[i+1]
// belong to system i (first may be null for one system).
template <typename T>
hipError_t chip_launch(int form, int kz, const ChipSys<T> *table, const int *first, int nsys, int tiles, hipStream_t s);

}  // namespace pfk
