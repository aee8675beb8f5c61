"""Problems that linear_bf16.hip's kernels take in both directions with the gate:
(H, T, D, rope_dim, rows aligned). tests/test_linear_workspace.py checks that they
do, so that a change of the routing rule does not drop them silently."""
BF16_KERNELS = [
    (2, 150, 32, 0, True), (2, 150, 32, 24, True), (1, 64, 32, 30, True), (2, 130, 32, 32, False), (2, 150, 32, 30, False),
    (2, 17 * 64 + 5, 64, 0, True), (1, 17 * 64 + 5, 64, 30, True), (2, 17 * 64 + 5, 64, 60, True),
    (1, 17 * 64 + 5, 64, 64, True), (2, 17 * 64 + 5, 64, 60, False), (1, 17 * 64 + 5, 64, 64, False),
    (10, 17 * 64 - 3, 128, 0, True), (10, 17 * 64 - 3, 128, 80, True), (10, 17 * 64 - 3, 128, 128, True),
    (10, 17 * 64 - 3, 128, 80, False),
]
