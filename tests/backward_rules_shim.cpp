// The host rules of the backward launch that choose between kernels, for the tests that hold them to what they are there for.
#include "tac_internal.h"

extern "C" int clear_in_recurrence(long long threads, long long floats) { return tac::backward_clear_in_recurrence((size_t)threads, (size_t)floats); }
