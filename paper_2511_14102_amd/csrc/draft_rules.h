// Which workgroups a draft launch is made of: rules on sizes alone, plain C++ (host code and kernels share them, and the
// CPU tests compile them by themselves).
#pragma once

namespace moespeq {

// Workgroups that reduce the router rows, the first ones of the launch, `rows` rows at a time each, for all tokens.  All workgroups
// wait for them, so calls on several streams that are dispatched together, each on its part of the units, go on only if one of
// them has all of these running: few of them, however many tokens there are.  (A row's tokens shared out over up to the whole
// grid shortened the start of a call, qwen3 shape, 8 tokens, 128 / 256 workgroups 37.5 / 36.5 us, and let two such calls wait for each other
// until their polls ran out.)
constexpr int router_workgroups(int E, int rows, int workgroups) {
    const int n = (E + rows - 1) / rows;
    return n < workgroups ? n : workgroups;
}

}  // namespace moespeq
