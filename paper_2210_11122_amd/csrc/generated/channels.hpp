// Generated by paper_2210_11122_amd.gen; do not edit.
// The amplitudes whose squares are the channel weights, in the order of the kernels: Feynman diagram and
// colour weight of each.
#pragma once
namespace me {
namespace rec2 {
constexpr int channel_diagram[3] = {0, 1, 2};
constexpr double channel_weight[3] = {5.333333333333333, 5.333333333333333, 12.0};
}
namespace rec3 {
constexpr int channel_diagram[18] = {0, 1, 3, 4, 6, 7, 2, 5, 8, 11, 10, 9, 13, 14, 12, 15, 15, 15};
constexpr double channel_weight[18] = {7.111111111111111, 7.111111111111111, 7.111111111111111, 7.111111111111111, 7.111111111111111, 7.111111111111111, 16.0, 16.0, 16.0, 16.0, 16.0, 16.0, 36.0, 36.0, 36.0, 36.0, 36.0, 36.0};
}
}  // namespace me
