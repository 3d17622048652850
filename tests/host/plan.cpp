// The tile choice of a batch (batch_plan), for tests that state which tiles
// they run.
#include "common.h"

extern "C" void plan(int wk, int pairs, int n_experts, int d_ff, int n_cu, int *align, int *list2) {
  const cep::BatchPlan p = cep::batch_plan(wk, pairs, n_experts, 2 * d_ff, n_cu);
  *align = p.align;
  *list2 = p.list2;
}
