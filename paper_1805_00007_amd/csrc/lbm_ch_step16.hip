// The population step with 16-bit storage (half and bfloat16 codes of g_i / w_i): the
// kernels of lbm_ch_step.hip instantiated for those storage modes only, in a translation
// unit of their own so that they can be built with machine-level loop-invariant code motion
// off (-mllvm -disable-machine-licm, see build.py), which would keep loop-invariant values
// in registers that the 16-bit decode needs.
#define LBM_STEP_16BIT_TU 1
#include "lbm_ch_step.hip"
