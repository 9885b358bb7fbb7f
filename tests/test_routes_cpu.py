"""The routing rules on boxes whose launches of several steps were measured
slower, or much faster, than one-step launches."""
import pytest

import routes

D3Q19, D3Q27 = 1, 2


# us per step, one-step against two-step launches.
@pytest.mark.parametrize("box", [
    (D3Q19, (512, 3, 512), "f64", (0, 1, 0), False, True),      # 19.2, 52.0
    (D3Q19, (512, 512, 4), "f64", (0, 0, 1), False, False),     # 29.7, 70.3
    (D3Q27, (512, 512, 4), "f64", (0, 0, 1), False, False),     # 40.8, 87.1
    (D3Q19, (512, 1, 512), "f64", (0, 0, 0), False, False),     # 15.3, 21.1
    (D3Q27, (112, 112, 112), "f64", (0, 0, 1), True, False),    # 98.6, 121.8
    (D3Q27, (160, 160, 160), "f64", (0, 0, 1), True, False),    # 288.3, 332.3
    (D3Q19, (160, 160, 160), "f32", (0, 0, 1), True, False),    # 104.9, 126.0
    (D3Q19, (160, 160, 160), "f32", (0, 3, 0), False, True),    # 100.4, 117.2
    (D3Q19, (512, 512, 4), "f32", (0, 0, 0), False, True),      # 28.7, 35.0
    (D3Q27, (128, 128, 128), "f32", (0, 1, 0), False, False),
    (D3Q19, (32, 256, 256), "f64", (0, 0, 0), False, False),
], ids=str)
def test_boxes_that_two_step_launches_would_slow_down(box):
    assert routes.march(*box) is None


@pytest.mark.parametrize("box", [
    (D3Q19, (256, 256, 256), "f64", (0, 0, 0), False, False),   # 812, 466
    (D3Q19, (512, 128, 128), "f64", (0, 1, 0), False, False),   # 400, 267
    (D3Q27, (512, 128, 128), "f64", (0, 1, 0), True, False),    # 578, 410
    (D3Q27, (512, 128, 128), "f64", (0, 0, 0), False, False),
    (D3Q19, (193, 127, 101), "f32", (0, 0, 0), False, True),    # 109, 78
    (D3Q19, (512, 3, 512), "f64", (0, 0, 0), False, False),     # 40.9, 32.3
    (D3Q19, (512, 512, 8), "f64", (0, 0, 0), False, False),     # 106, 80
    (D3Q19, (64, 64, 64), "f64", (0, 0, 0), False, False),      # 15.5, 14.5
], ids=str)
def test_boxes_that_two_step_launches_speed_up(box):
    assert routes.march(*box)
