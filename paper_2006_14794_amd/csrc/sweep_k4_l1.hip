// Sweep kernel instantiations: lifted forward (Gaussian static kernel), dyadic order 1 (see sweep_inst.h).
#define SK_KIND 4
#define SK_LAM 1
#define SK_NG 1
#include "sweep_inst.h"
