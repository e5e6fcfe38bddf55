// Sweep kernel instantiations: forward with the implicit scheme's cell factor, dyadic order 3 (see sweep_inst.h).
#define SK_KIND 5
#define SK_LAM 3
#define SK_NG 1
#include "sweep_inst.h"
