// The bunch kernel's builds for inclined rays outside the moment series and for the
// curved atmosphere, compiled apart from the rest: the reason and the figures stand
// with their list at the end of the bunch kernel.
#define CKV_SLOWPATH
#include "ckv_kernels.hip"
