#define SK_LAM 1
#define SK_ROWS 8
#define SK_NG 4
#include "grad_rev_inst.h"
