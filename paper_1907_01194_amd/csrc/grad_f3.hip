// The spin-3 instances of the fused energy / gradient x pass.
#define GPE_GRAD_F 3
#include "grad_x.h"
