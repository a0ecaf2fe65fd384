// NEP forces of small systems (nep_small.hip).
#pragma once

#include "internal.hpp"
#include "nep_kernels.hpp"

namespace nep {

// Whether a call of P beads and `rows` = P N (bead, atom) rows takes the
// one-wavefront-per-row kernels.  Both forms give the same bits, so the line
// follows the time alone: the general kernels take one walk over a lane's
// lists, however few rows there are, these kernels a time that grows with
// the rows and little with the lists.  slots: candidate capacities of a row,
// radial + angular, which the callers fit to the longest rows.  us of
// nep_compute by the general / these kernels, [slots]:
//   vector network, one species: FCC metal (4, 4) 1 bead 6,144 rows [80]
//   94 / 68, 8,192 [81] 97 / 90, 12,288 [81] 102 / 132; 4 beads 8,192 [93]
//   81 / 79, 12,288 [97] 82 / 112; 8 beads 12,288 [106] 84 / 83; 32 beads
//   [109] 80 / 77; cutoffs (6, 5) instead of (5, 4) 1 bead 12,288 [145] 154 /
//   148; at a quarter of its density 4 beads 4,096 [47] 48 / 43,
//   6,144 [38] 48 / 52, 8 beads 8,192 [47] 47 / 52; (8, 8) 1 bead 12,288
//   [145] 243 / 201, 32 beads [166] 201 / 141;
//   several species: water 1 bead 12,288 [168] 296 / 160, 8 beads 157 / 109;
//   thin water 1 bead 8,192 [52] 113 / 90, 12,288 [52] 122 / 130; 64 beads
//   8,192 [63] 55 / 54, 12,288 [57] 60 / 72; framework (8, 6) 1 bead 12,288
//   [43] 175 / 152, 64 beads 8,192 [49] 83 / 79, 12,288 [47] 90 / 97;
//   matrix-core network, whose 16-row tile holds one row here: (4, 4) 1 bead
//   metal 6,144 [80] 93 / 79, 9,216 100 / 122, with rows twice as long 143 /
//   135, 8 beads 12,288 117 / 132; (8, 8) 1 bead 6,144 [143] 211 / 167, 9,216
//   209 / 254, thin 3,072 [33] 81 / 80, 4,096 [32] 82 / 102; framework 1 bead
//   6,144 [43] 144 / 122, 32 beads [47] 116 / 102, 64 beads 4,096 [47] 61 /
//   62, 6,144 [46] 73 / 114, at a third of its density 1 bead 4,096 [18] 72 /
//   65, 6,144 [21] 82 / 98.
constexpr int64_t kSmallRows = 12288, kSmallRowsFew = 8192, kSmallRowsMf = 6144;
inline bool takes_small(int64_t rows, int P, const nep_hparams &h, int slots, int mlp)
{
    const bool vec = mlp == NEP_MLP_FP32;
    const int S = h.n_species;
    // few beads (gathers that share few cache lines) against the general
    // kernels' shortest walks: one species, few angular functions, short cutoffs
    const bool few = P < 8 && S == 1 && h.n_max_angular + 1 <= 5 && h.rc_angular < 4.6;
    const int64_t most = !vec ? kSmallRowsMf : few ? kSmallRowsFew : kSmallRows;
    // lists below `full` slots shorten the general kernels' walk in proportion
    // (more than 32 beads: one atom per wavefront, whose walk is shorter)
    const int full = vec ? (S == 1 ? 76 : P > 32 ? 90 : 64) : (S == 1 ? 90 : P > 32 ? 80 : 40);
    return rows * full <= most * (slots < full ? slots : full);
}
constexpr int kRowValues = 19;   // per row: site energy, 9 angular and 9 radial virial entries

int32_t launch_small(const NepArgs &a, const nep_model *m, const int32_t *atom_sys, float *rowp, hipStream_t s);

}  // namespace nep
