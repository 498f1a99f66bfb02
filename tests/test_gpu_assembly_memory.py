"""Device memory that the assembly of E takes and gives back: E, and the phase
matrix with the planes of the split k range (together at most 2.5 E or 128
MiB), watched from another thread during builds in a row. More than that made
builds in a row wait for the driver to clear what they had released.
"""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MB = 1 << 20


@pytest.mark.parametrize("n", [1000, 2048, 4096, 4608])
def test_transient_memory(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_06704_amd import cpm
    box = np.array([39.4, 51.1, 100.0])
    pos = np.random.default_rng(1).random((n, 3)) * box
    cpm.System(pos, box).close()   # loads the code
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    least, stop = [free], threading.Event()

    def watch():
        while not stop.is_set():
            least[0] = min(least[0], torch.cuda.mem_get_info()[0])

    t = threading.Thread(target=watch)
    t.start()
    try:
        for _ in range(20):
            cpm.System(pos, box).close()
    finally:
        stop.set()
        t.join()
    e = 8.0 * ((n + 127) // 128 * 128) ** 2
    used = free - least[0]
    print(f"[case] N={n}: {used / MB:.0f} MB, E {e / MB:.0f} MB", flush=True)
    # 32 MB for the k-set, positions and tables, and the allocator's pages
    assert used <= e + max(2.5 * e, 128 * MB) + 32 * MB
