"""How the attention's cost line is shared out, on the host: the functions of the kernel in a small program of their own."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2510_27641_amd import build

PROGRAM = """
#include "attn_mfma_kernel.h"
#include <cstdio>
int main()
{
    using namespace specattn;
    int total, n_wg, rows;
    while (std::scanf("%d %d %d", &total, &n_wg, &rows) == 3) {
        for (int w = 0; w < n_wg; ++w) {
            const auto s = make_share<32>(total, n_wg, rows, w);
            std::printf("%d %d %d ", s.c0, s.c1, share_index(w, n_wg));
        }
        std::printf("\\n");
    }
}
"""


@pytest.fixture(scope="module")
def shares(tmp_path_factory):
    if not (shutil.which(build.HIPCC) or os.path.exists(build.HIPCC)):
        pytest.skip("hipcc is missing")
    folder = tmp_path_factory.mktemp("shares")
    src, exe = folder / "shares.hip", folder / "shares"
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, *build.FLAGS, "--offload-host-only", str(src), "-o", str(exe)], check=True)

    def ask(questions):
        lines = "".join("%d %d %d\n" % q for q in questions)
        out = subprocess.run([str(exe)], input=lines, capture_output=True, text=True, check=True).stdout.splitlines()
        return [np.array(line.split(), dtype=np.int64).reshape(-1, 3) for line in out]
    return ask


@pytest.mark.parametrize("n_wg", [32, 38, 64, 128, 256, 304])
def test_the_line_is_shared_out_whole(shares, n_wg):
    """Shares follow each other without gaps, none is empty ahead of the line's end, every one has an owner.  They are equal but
    for one unit, or - of 32 tiles and more, on a whole GPU of eight XCDs - but for the tilt, which leaves every second boundary in its place."""
    rng = np.random.default_rng(n_wg)
    totals = [0, 1, n_wg - 1, n_wg, n_wg + 1, 1000 * n_wg, 1000 * n_wg + 5, 2 ** 22 - 3]
    questions = [(int(t), n_wg, rows) for rows in (1, 64, 128, 256, 1536)
                 for t in totals + [32 * n_wg + 12 * rows + k for k in (-1, 0, 1)] + list(rng.integers(1, 400 * n_wg, size=20))]
    for (total, _, rows), s in zip(questions, shares(questions)):
        begin, end, owner = s.T
        assert begin[0] == 0 and end[-1] == total and np.array_equal(begin[1:], end[:-1])
        size = end - begin
        assert (size[:min(n_wg, total)] > 0).all() and (size[min(n_wg, total):] == 0).all()
        assert np.array_equal(np.sort(owner), np.arange(n_wg))
        exact = np.arange(n_wg + 1) * total // n_wg if total >= n_wg else np.minimum(np.arange(n_wg + 1), total)
        bounds = np.append(begin, total)
        tilted = n_wg == 256 and total - 12 * rows >= 32 * n_wg and (2 * rows <= n_wg or total % n_wg != 0)
        assert np.array_equal(bounds[::2], exact[::2])
        assert np.array_equal(bounds, exact) != tilted
        assert np.abs(bounds - exact).max() <= (total / n_wg * 5 / 128 + 1 if tilted else 0)
