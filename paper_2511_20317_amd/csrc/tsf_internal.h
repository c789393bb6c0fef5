// tsf_internal.h -- helpers shared by the translation units of libtsf.
#pragma once
#include "../../include/tsf.h"

// Record the reason of an error for tsf_last_error() and return `st`.
tsf_status tsf_fail(tsf_status st, const char *fmt, ...) __attribute__((format(printf, 2, 3)));

// tsf_mlp_fwd whose hidden layers are not written where h1 or h2 is null.
tsf_status mlp_forward(const tsf_mlp *net, const uint16_t *X, int32_t M, uint16_t *h1,
                       uint16_t *h2, float *logit, void *hip_stream);
