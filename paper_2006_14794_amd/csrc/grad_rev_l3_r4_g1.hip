#define SK_LAM 3
#define SK_ROWS 4
#define SK_NG 1
#include "grad_rev_inst.h"
