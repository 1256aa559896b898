// Host builder of the mechanism tables the wave-per-cell integrator reads.
//
// The wave kernel gives every lane an equal share of the work of a cell's
// right-hand side and Jacobian, so the tables are laid out lane by lane:
// entry (i, lane) of a table at [i * 64 + lane], one coalesced load per i.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>
#include <vector>

#include "chem_internal.h"

namespace chem {

// Reaction words: the four species slots, 6 bits each (K, at most 63, marks
// an empty slot), the pressure-dependence kind in bits 24..26 and the
// irreversible flag in bit 31.
constexpr uint32_t kRxnWordIrrev = 0x80000000u;

// Device tables of one mechanism (pointers into its device block).
//
// Scratch of the kernel, in doubles: slot 0 holds 0 (the target of padded
// entries), then for the production sums +v_r at 1 + r and -v_r at 1 + R + r,
// for the Jacobian the four slot derivatives of reaction r at 1 + 4 r.
struct Wave64Tables {
    int32_t rounds;            // reactions per lane in the tables, max(4, ceil(R / 64))
    int32_t gather4;           // production entries per lane / 4
    int32_t extras;            // most extra segments of one species
    int32_t jrounds;           // Jacobian entries per lane
    const double2 *rx;         // [rounds][2][64]: (ln A, b), (Ea / Ru, change of moles); padded ones have rate 0
    const uint32_t *rw;        // [rounds][64]: reaction words
    // production of the species: lane k < K sums the first entries of species
    // k, lanes from K on the entries of species with more than 4 gather4;
    // byte offsets into the scratch (a coefficient of 2 is two entries)
    const uint4 *gat;          // [gather4][64]
    const int32_t *xseg;       // [64]: species k's extra lanes, first | count << 8
    // non-zero entries of the species block of the Jacobian, most
    // contributions first; contribution: byte offset | sign << 31
    const int2 *jcnt;          // [jrounds]: offset of the round's contributions / 64, contributions per lane (of 4)
    const uint32_t *jrc;       // [jrounds][64]: row | column << 8, 0xFFFF for a padded entry
    const uint32_t *jcon;      // contributions, [offset][64]
    // NASA-7 blocks, [2 ranges][7][64] pairs of coefficients
    const double2 *th;
    const double *tmid;        // [64]
    const double *invw;        // [64]: 1 / W_k, 0 beyond the species
    // pressure-dependent reactions of species k: entries pent[poff[k] .. poff[k+1]) of (reaction, net coefficient)
    const int32_t *poff;       // [65]
    const int2 *pent;
};

// Builds the tables for K species and the reactions rx (inc[k]: the
// (reaction, net coefficient) pairs of species k, in reaction order; species:
// K blocks of kSpeciesLen; W: kg/mol; aux: the records of the pressure-dependent
// reactions).  Returns the bytes to place 256-byte aligned in
// device memory at address `base`; t receives the pointers.
std::vector<char> build_wave_tables(int K, const std::vector<DevRxn> &rx, int R,
                                    const std::vector<std::vector<std::pair<int, int>>> &inc,
                                    const std::vector<double> &species, const std::vector<double> &W,
                                    const std::vector<double> &aux, const char *base, Wave64Tables &t);

}  // namespace chem
