// The LM head's argmax (lm_head.hip) as the greedy acceptance launches it.
#pragma once
#include <hip/hip_runtime.h>

struct alignas(8) LmBest { float v; int i; };   // best logit of some tokens and the token (the smallest of equals); none: { -inf, INT_MAX }

// How the vocabulary is shared out: `chunks` shares of `share` tokens, for one of three arrangements of a workgroup's waves.
enum LmForm { LM_FEW, LM_TALL, LM_WIDE };
struct LmShares { LmForm form; int vt, share, chunks; };

LmShares lm_shares(int R, int V);                       // R rows of hidden states; no more than ceil(V / 32) chunks

// part[chunk * R + row]: the best of a share's tokens for every row
int lm_head_launch(const LmShares &p, const void *H, const void *W, int R, int h, int V, LmBest *part, hipStream_t st);
