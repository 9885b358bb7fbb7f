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


def test_every_launch_makes_steps_that_its_kernel_can():
    """Over boxes, storages, walls and step counts: the launches add up to the
    steps, none makes more steps than its regions or strips can, and strips of
    eight run only where they are built (periodic, FP64 and FP32)."""
    can = {"24x8": 8, "32x8": 8, "32x6": 6, "32x4": 4, "one": 1}
    dims = [(1, 1), (7, 5), (128, 128), (130, 97), (16, 4096), (260, 250), (300, 270), (700, 700), (65000, 3),
            (1024, 1024), (1448, 1448), (1500, 1400), (2048, 2048), (2100, 2000), (2900, 2900), (4096, 4096),
            (65535, 32767)]
    questions = [(d, st, walls, mask, comp, steps) for d in dims for st in routes.STORAGE
                 for walls, mask in ((0, 0), (1, 0), (1, 1)) for comp in (0, 1) for steps in range(1, 30)]
    for q, launches in zip(questions, routes.boxes_2d(questions)):
        d, st, walls, mask, comp, steps = q
        assert sum(k for k, _ in launches) == steps, q
        for k, kind in launches:
            if kind == "strips":
                assert k == 4 or (k == 8 and not walls and st in ("f64", "f32")), q
            else:
                assert k <= can[kind], q


# us per step, one-step against the launches of several steps.
@pytest.mark.parametrize("q", [
    ((65000, 3), "f64", True, False, False, 48),     # 7.8, 11.5
    ((65000, 3), "f16", True, False, True, 48),      # 4.1, 14.4
    ((2048, 2048), "f16", True, False, False, 48),   # 30.4, 34.8
    ((1024, 1024), "f16", True, False, True, 48),
    ((1024, 1024), "f16", False, False, False, 3),   # 9.6, 13
    ((512, 512), "f16", True, False, True, 2),       # 5.3, 6.8
    ((1024, 1024), "e4m11", False, False, False, 48),  # 9.5, 12.1
    ((2048, 2048), "e4m11", False, False, False, 48),  # 26.7, 46.9
    ((1024, 1024), "e4m11", True, False, False, 48),   # 11.9, 13.4
    ((512, 512), "e4m11", False, False, False, 5),     # 4.6, 5.6
    ((512, 512), "f32", True, False, True, 2),
    ((16, 65000), "f16", True, False, True, 48),       # 11.3, 15.1
    ((16, 65000), "e4m11", True, True, False, 48),     # 14.5, 17.4
    ((65000, 16), "f32", True, False, True, 2),        # 17.1, 20.1
], ids=str)
def test_boxes_that_2d_launches_would_slow_down(q):
    assert all(kind == "one" for _, kind in routes.boxes_2d([q])[0])


@pytest.mark.parametrize("q,launches", [
    (((128, 128), "f64", False, False, False, 19), [(8, "24x8"), (8, "24x8"), (3, "24x8")]),
    (((128, 128), "e4m11", True, False, True, 10), [(8, "24x8"), (2, "24x8")]),
    (((512, 128), "f64", True, True, False, 10), [(8, "32x8"), (2, "32x8")]),
    (((700, 700), "f32", False, False, False, 14), [(6, "32x6"), (4, "32x4"), (4, "32x4")]),
    (((512, 512), "f16", True, False, False, 14), [(6, "32x6"), (4, "32x6"), (4, "32x6")]),
    (((512, 512), "e4m11", False, False, False, 8), [(6, "32x6"), (1, "one"), (1, "one")]),
    (((4096, 4096), "f64", False, False, False, 13), [(8, "strips"), (4, "32x4"), (1, "one")]),
    (((4096, 4096), "f16", False, False, False, 7), [(4, "strips")] + 3 * [(1, "one")]),
    (((2000, 1600), "bf16", True, True, False, 9), [(4, "strips"), (4, "strips"), (1, "one")]),
], ids=str)
def test_2d_launches(q, launches):
    assert routes.boxes_2d([q])[0] == launches
