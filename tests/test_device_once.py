"""Set-up that is due once per device: every device gets its own, a failure is
reported and tried again, and what is done is not repeated."""
from host_rules import run_program

BODY = """
    static lx::DeviceOnce once;
    static int calls = 0;
    int device, result;
    std::cin >> device >> result;
    const int got = once.run(device, 0, [&] { ++calls; return result; });
    std::printf("%d %d\\n", got, calls);
"""


def test_device_once(tmp_path):
    steps = [  # device, what the set-up returns -> returned, calls so far
        ((0, 7), (7, 1)), ((0, 0), (0, 2)), ((0, 7), (0, 2)),
        ((1, 0), (0, 3)), ((1, 7), (0, 3)), ((63, 7), (7, 4)), ((63, 0), (0, 5)), ((63, 7), (0, 5)),
        ((64, 0), (0, 6)), ((64, 7), (7, 7)), ((-1, 0), (0, 8)), ((0, 7), (0, 8)),
    ]
    rows = run_program(tmp_path, "lx_device_once.h", BODY, [s for s, _ in steps])
    assert [tuple(map(int, r)) for r in rows] == [want for _, want in steps]


def test_no_attribute_is_set_once_per_process():
    """Kernel attributes belong to the device that is current: no `static`
    result of hipFuncSetAttribute."""
    import glob
    import os
    import re
    from paper_2608_07814_amd import build as B
    for path in glob.glob(os.path.join(B.CSRC, "*.hip")):
        src = open(path).read()
        assert not re.search(r"static\s+(const\s+)?hipError_t\s+\w+\s*=", src), path
