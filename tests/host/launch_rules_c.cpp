// C names for the launch rules (launch_rules.h), for tests/test_launch_rules.py.
#include "launch_rules.h"

using namespace mics;

extern "C" {
size_t rules_lds(int lanes, int waves_per_cu, size_t needed) { return lds_for(Shape{lanes, waves_per_cu}, needed); }
}
