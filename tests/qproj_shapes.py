"""Projections of pseudo queries by the plan that they get: (layers, heads, head size, rows, hidden) -> waves of a workgroup, planes of
partial sums.  tests/test_qproj_plan.py holds the list to the planner; the GPU tests run the shapes."""
SPLIT_SHAPES = {
    (5, 8, 128, 32, 8192): (1, 16),     # 65 to 80 tiles of 64 features against 8192 channels: single waves stay, each with a plane
    (6, 9, 72, 7, 8192): (1, 16),
    (1, 36, 128, 16, 8192): (1, 16),
}
