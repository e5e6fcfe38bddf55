#define SK_LAM 0
#define SK_ROWS 4
#define SK_NG 4
#include "grad_rev_inst.h"
