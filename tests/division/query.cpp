// The host rules that divide launches (csrc/fa_launch.h), for tests that have to know which division a shape takes.
#include "../../paper_2407_08608_amd/csrc/fa_launch.h"

extern "C" int key_split(int fp8, long heads, int N, int d, int causal) {
    return fp8 ? fa::few_forward_fp8(heads, N, d, causal) : fa::few_forward(heads, N, d, causal);
}

// "large", "keys32", "one32", "rows behind" or "rows ahead" (of the key blocks)
extern "C" const char* backward_form(long heads, long kv_heads, int N, int d, int causal) {
    switch (fa::choose_bwd_form(heads, kv_heads, N, d, causal)) {
        case fa::kBwdLarge: return "large";
        case fa::kBwdKeys32: return "keys32";
        case fa::kBwdOne32: return "one32";
        default: return fa::bwd_rows_first(heads / kv_heads, causal) ? "rows ahead" : "rows behind";
    }
}

extern "C" int backward_own_row_sums(long heads, long kv_heads, int N, int d) { return fa::bwd_own_row_sums(heads, kv_heads, N, d); }
