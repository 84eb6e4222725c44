// Record of the stubbed launches (host sanitizer build of the host layer).
#pragma once
#include <stddef.h>

#include <hip/hip_runtime_api.h>

struct StubLog {
  int attn_bf16 = 0, attn_f32 = 0, merge = 0, accept = 0, sample = 0, tree_calls = 0, commit = 0;
  int entropy = 0, entropy_steps = 0;  // calls with the root entropy; of these, workgroups of several steps
  int nsplit = 0;                      // splits of the last fp32 attention
  bool tree = false;
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  const void* ws = nullptr;  // the workspace the next call receives
  size_t ws_bytes = 0;
};
extern StubLog g_stub;
