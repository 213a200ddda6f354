// Slab GEMMs with fp16 W (gemm_slab.h), one kernel per row of the table in
// gemm_common.h, epilogue and layout.
#include "gemm_slab.h"

namespace pipo {

void launch_slab_f16(const GemmArgs& a, int epi, int idx, bool direct, int S, float* ws,
                     hipStream_t st) {
  switch (idx) {
#define PIPO_CASE(i, MF, NF, WN, KS, PD) \
  case i: return launch_slab<MF, NF, WN, KS, PD, false>(a, epi, direct, S, ws, st);
    PIPO_SLAB_F16(PIPO_CASE)
#undef PIPO_CASE
  }
}

}  // namespace pipo
