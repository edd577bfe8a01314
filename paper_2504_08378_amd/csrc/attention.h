// Arguments of the decode attention, shared by the attention launches (attention.hip) and the
// attention phase of the whole-layer kernel (layer.hip).
#pragma once
#include "af_internal.h"

struct AttnParams {
  const half_t* qkv;   // [q | k | v] of the new token, before rotation
  half_t* k_cache;     // [n_kv][cap][HD]
  half_t* v_cache;
  half_t* out;         // [n_heads*HD]
  float* part;         // [n_heads][KS][HD+2]
  int* tickets;
  int ticket0;         // this token's first ticket
  int group_heads;     // query heads of a workgroup, at most 8
  int n_heads, n_kv, kv_len, kv_cap, head_dim;
  long long* prof;     // time stamps of this launch (af_profile_set), or null
  float cs[64], sn[64];  // cos / sin of pos * theta^(-2i/HD), i < HD/2, formed in fp64 on the host
};
