// The integer kernels of the gfx950 Catalan library and its C ABI in one
// translation unit, so that the __constant__ tables need no relocatable device
// code (the FP64 transforms, with constants of their own, are fntt.hip).
#include "common.hpp"
#include "fntt.hpp"
#include "ntt.inc.hip"
#include "small.inc.hip"
#include "fused.inc.hip"
#include "sieve.inc.hip"
#include "ratio.inc.hip"
#include "decimal.inc.hip"
#include "host.inc.hip"
#include "decimal_host.inc.hip"
#include "rates.inc.hip"
