#include "scratch_part.h"

SCRATCH_PART(2)
