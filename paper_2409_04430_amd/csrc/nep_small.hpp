// NEP forces of small systems (nep_small.hip).
#pragma once

#include "internal.hpp"
#include "nep_kernels.hpp"

namespace nep {

// Largest number of (bead, atom) rows that take the one-wavefront-per-row
// kernels.  Force calls (lists given), one lane per row against one
// wavefront per row, us: FCC metal 864 rows 97 / 26, 6,912 rows 101 / 56,
// 16,384 rows 100 / 110; water 6,144 rows 146 / 59, 12,288 rows 188 / 109,
// 24,576 rows 177 / 197.  With a matrix-core network, whose 16-row tile
// holds one row here: four-body shape (8, 8) 6,000 rows 222 / 153, 10,368
// rows 231 / 265; (8, 6) 3,456 rows 110 / 82, 11,664 rows 163 / 224; (4, 4)
// 10,368 rows 137 / 109.  Both forms give the same bits.
constexpr int64_t kSmallRows = 12288, kSmallRowsMf = 6144;
inline bool takes_small(int64_t rows, int mlp) { return rows <= (mlp == NEP_MLP_FP32 ? kSmallRows : kSmallRowsMf); }
constexpr int kRowValues = 19;   // per row: site energy, 9 angular and 9 radial virial entries

int32_t launch_small(const NepArgs &a, const nep_model *m, const int32_t *atom_sys, float *rowp, hipStream_t s);

}  // namespace nep
