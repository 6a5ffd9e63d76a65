// Between this library and the binding's native wrappers; not part of the C ABI.
#pragma once

#include "specsteer.h"

// specsteer_verify_block for a caller whose host time is small beside the GPU's: rows without drafts are shaped for the GPU's time
// alone, as under stream capture.
extern "C" ss_status specsteer_verify_block_unbound(const void* G, const void* S_ctx, const void* S_noctx, const int32_t* draft,
                                                    const int32_t* draft_len, const float* uniforms, const ss_params* params,
                                                    int32_t* accepted_len, int32_t* next_token, float* next_token_logprob,
                                                    float* recovery_logprobs, float* draft_logprobs, void* workspace,
                                                    size_t workspace_bytes, void* stream);
