// The library's host rules and index arithmetic, callable from the tests (tests/test_host_rules.py).
#include "prefill_shape.hpp"

using namespace optgqa;

extern "C" int prefill_shape_of(int64_t units8, int shift, int max_q_len, int windowed, int whole_prompts, int cus)
{
    return (int)prefill_shape(units8, shift, max_q_len, windowed, whole_prompts, cus);
}
