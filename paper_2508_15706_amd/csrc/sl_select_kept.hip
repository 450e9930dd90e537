// Kernel A of sl_compress for lists whose rows are not aligned (a translation unit of its own: each takes over a minute to compile).
#include "sl_select_kernel.h"

void (*sl_select_kept(int k, bool two_bit, bool params))(SelectArgs) { return select_for<true>(k, two_bit, params); }
