// The resident CG's kernels in fp32 (a file of its own so that both precisions compile side
// by side).
#include "erc_resident.h"

namespace erc {

hipError_t res_solve_f32(const ResArgs& a, int ncols, size_t lds, hipStream_t s) {
  return res_dispatch<float>(a, ncols, lds, s);
}

}  // namespace erc
