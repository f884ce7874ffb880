// The spin-1 instances of the fused energy / gradient x pass.
#define GPE_GRAD_F 1
#include "grad_x.h"
