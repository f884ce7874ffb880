// The spin-2 instances of the fused energy / gradient x pass.
#define GPE_GRAD_F 2
#include "grad_x.h"
