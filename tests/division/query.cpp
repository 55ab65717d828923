// The host rules that divide forward launches (csrc/fa_launch.h), for tests that have to know which division a shape takes.
#include "../../paper_2407_08608_amd/csrc/fa_launch.h"

extern "C" int key_split(int fp8, long heads, int N, int d, int causal) {
    return fp8 ? fa::few_forward_fp8(heads, N, d, causal) : fa::few_forward(heads, N, d, causal);
}
