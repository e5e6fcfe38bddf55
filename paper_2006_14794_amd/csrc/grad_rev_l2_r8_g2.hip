#define SK_LAM 2
#define SK_ROWS 8
#define SK_NG 2
#include "grad_rev_inst.h"
