"""The walk of a grid over the elements of a launch, in block order and by
XCD: every element is taken once, and by XCD every region is consecutive and
no XCD gets more than its blocks' share.  Host code of the kernels' headers;
on the GPU the walks give the fused call's shares (integers: no tolerance)."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2309_04909_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"

DRIVER = '''
#include <stdio.h>
#include <vector>
#include "bc_device.h"
int main() {
    const unsigned grids[] = {1, 2, 7, 8, 9, 15, 16, 17, 63, 64, 100, 256};
    const unsigned counts[] = {1, 255, 256, 257, 2047, 2048, 2049, 5000, 16384, 16385, 20000, 30001, 65536, 70001, 200000};
    for (unsigned asked : grids)
        for (unsigned count : counts)
            for (int by_xcd = 0; by_xcd < 2; ++by_xcd) {
                const unsigned grid = bc::walk_grid(by_xcd, asked), chunks = (count + 255) / 256;
                std::vector<unsigned> seen(count, 0);
                unsigned wrong = 0, split = 0, more = 0, next = 0;
                for (unsigned x = 0; x < 8; ++x) {
                    unsigned lo = count, hi = 0, taken = 0;
                    for (unsigned b = x; b < grid; b += 8)
                        for (unsigned t = 0; t < 256; ++t) {
                            const bc::WalkRange r = bc::walk_range(by_xcd, b, t, grid, count);
                            for (unsigned i = r.begin; i < r.end; i += r.stride, ++taken) {
                                if (i >= count || seen[i]++) ++wrong;
                                if (i < lo) lo = i;
                                if (i >= hi) hi = i + 1;
                            }
                        }
                    if (by_xcd && taken && (hi - lo != taken || lo != next)) ++split;
                    if (taken) next = hi;
                    if (by_xcd && (taken + 255) / 256 > chunks / 8 + 1) ++more;
                }
                for (unsigned i = 0; i < count; ++i) wrong += seen[i] != 1;
                printf("%u %u %d %u %u %u\\n", asked, count, by_xcd, wrong, split, more);
            }
}
'''


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_every_element_once_and_balanced(tmp_path):
    src, exe = tmp_path / "walk.hip", tmp_path / "walk"
    src.write_text(DRIVER)
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O2", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    lines = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300).stdout.strip().split("\n")
    assert len(lines) == 12 * 15 * 2
    for line in lines:
        assert line.endswith(" 0 0 0"), "grid, elements, by XCD, taken not once, regions not consecutive, chunks above an eighth: " + line


@pytest.mark.gpu
@pytest.mark.parametrize("bpc", [1, 3])
@pytest.mark.parametrize("extra", [0, 1, 255, 32 * 77 + 9])
def test_strided_walks_match_the_fused_call(bpc, extra):
    """Grids that stride: 256 compute units at 1 and 3 blocks, ragged last strides, both forms of the planes."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_04909_amd import bicop as B
    prm, sd, n = B.Params(64, 18, 13), B.Seeds(11, 12, 13, 14), 5 * 65536 + extra
    gen = torch.Generator(device="cuda").manual_seed(n)
    x0, x1 = (torch.randint(-(1 << 62), 1 << 62, (n,), generator=gen, device="cuda") for _ in range(2))
    want = B.drelu(x0, x1, prm, sd)
    kinds = ("fused", "pre", "expand")
    before = {k: B.get_schedule(k, 19, 8, B.BC_OP_DRELU) for k in kinds}
    try:
        for k in kinds:
            B.set_schedule(k, 19, bpc, 8, B.BC_OP_DRELU)
        got = B.drelu_pre(x0, x1, prm, B.rand_expand(B.BC_OP_DRELU, prm, sd, n))
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        d = B.drelu_reply(B.drelu_send(0, x0, prm, sd), B.drelu_send(1, x1, prm, sd), prm, sd)
        assert torch.equal(B.drelu_finish(0, d[0], prm, sd), want[0])
        assert torch.equal(B.drelu_finish(1, d[1], prm, sd), want[1])
    finally:
        for k, v in before.items():
            B.set_schedule(k, 19, v, 8, B.BC_OP_DRELU)
