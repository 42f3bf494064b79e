"""Projections of pseudo queries by the plan that they get: (layers, heads, head size, rows, hidden) -> waves of a workgroup, planes of
partial sums.  tests/test_qproj_plan.py holds the list to the planner; the GPU tests run the shapes."""
SPLIT_SHAPES = {
    (3, 38, 72, 65, 1024): (1, 2),
    (3, 38, 72, 65, 2048): (1, 4),
    (8, 9, 72, 37, 5184): (1, 8),
    (6, 9, 72, 65, 1024): (4, 1),
    (4, 32, 128, 64, 1024): (4, 1),
    (1, 1, 64, 7, 1024): (4, 2),
    (1, 2, 72, 7, 2112): (4, 3),
    (2, 5, 72, 37, 2048): (4, 4),
    (8, 2, 72, 65, 4160): (4, 5),
    (1, 3, 72, 37, 4160): (4, 6),
    (1, 3, 72, 37, 4672): (4, 7),
    (1, 3, 72, 37, 4096): (4, 8),
    # 65 to 80 tiles of 64 features against 8192 channels: single waves would have sixteen planes
    (5, 8, 128, 32, 8192): (4, 3),
    (6, 9, 72, 7, 8192): (4, 3),
    (1, 36, 128, 16, 8192): (4, 3),
}
