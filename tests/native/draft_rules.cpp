// The size rules of the draft calls (csrc/draft_rules.h) for ctypes.
#include "draft_rules.h"

using namespace moespeq;

extern "C" {

int rule_router_workgroups(int experts, int rows, int workgroups) { return router_workgroups(experts, rows, workgroups); }

}
