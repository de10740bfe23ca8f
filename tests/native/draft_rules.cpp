// The size rules of the draft calls (csrc/draft_rules.h) for ctypes.
#include "draft_rules.h"

using namespace moespeq;

namespace {
Shape one_token(int H, int E, int I, int k, int g, int S) { return Shape{1, H, E, I, k, S, g, 1}; }
}

extern "C" {

int rule_router_workgroups(int experts, int rows, int workgroups) { return router_workgroups(experts, rows, workgroups); }
int rule_fits(int H, int E, int I, int k, int g, int S, int tokens) { return draft_fits(one_token(H, E, I, k, g, S), tokens, false); }
int rule_shared_inside(int H, int E, int I, int k, int g, int S, int n_cu) { return draft_shared_inside(one_token(H, E, I, k, g, S), n_cu); }
// 0: single items, 1: pairs, 2: the persistent launch
int rule_one_token_form(int H, int E, int I, int k, int g, int S, int shared_inside, int n_cu, int single_slots)
{
    return one_token_form(one_token(H, E, I, k, g, S), false, shared_inside != 0, n_cu, [=] { return single_slots; });
}

}
