"""The rule by which the planes of records and messages go through the L2 or
around it: small planes and large ones of whole 128-byte lines go around it,
and a reader never goes through the L2 where the writer went around it.  The
rule is host code of the kernels' headers; on the GPU both forms give the fused
call's shares on each side of every limit (integers: no tolerance)."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2309_04909_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"
MIB = 1 << 20

DRIVER = '''
#include <stdio.h>
#include "internal.h"
int main() {
    unsigned long long at, n, bytes, messages;
    while (scanf("%llu %llu %llu %llu", &at, &n, &bytes, &messages) == 4)
        printf("%d %d\\n", (int)bc::planes_around_l2((const void*)at, n, bytes, messages),
               (int)bc::planes_cached((const void*)at, n, bytes, messages));
}
'''


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_rule(tmp_path):
    # (address, elements, bytes an element): (written around the L2, read through it)
    whole = {
        (256, 1 << 18, 56): (1, 0), (256, 1 << 18, 216): (1, 0), (256, 1 << 19, 72): (1, 0),       # small
        (256, 1 << 20, 56): (1, 0), (256, (1 << 20) + 32, 56): (0, 1),                             # 56 MiB and above
        (256, 1 << 20, 124): (0, 1), (256, 1 << 20, 264): (0, 1), (256, (1 << 20) + 32, 264): (0, 0),
        (256, 1 << 21, 288): (0, 0), (256, (1 << 21) + 32, 288): (1, 0), (256, (1 << 21) + 32, 100): (0, 1),
        (256, (1 << 21) - 32, 8): (1, 0), (256, 1 << 21, 8): (0, 1), (256, 1 << 21, 16): (0, 1),   # few bytes each
        (256, (1 << 21) - 32, 16): (1, 0), (256, 1 << 22, 8): (0, 1), (256, 1 << 26, 8): (1, 0),
        (256, 1 << 22, 80): (1, 0), (256, 1 << 23, 132): (1, 0),                                   # above the cache
    }
    shared = {                                                            # of a record, of messages
        (256, (1 << 18) + 1, 56): ((0, 1), (1, 0)), (256, (1 << 18) + 1, 64): ((0, 1), (0, 1)),
        (256, 1000003, 124): ((0, 1), (0, 1)), (256, 4000003, 124): ((0, 0), (0, 0)),
        (16, 1 << 18, 216): ((0, 1), (0, 1)), (16, 1 << 23, 132): ((0, 0), (0, 0)), (16, 1 << 18, 60): ((0, 1), (1, 0)),
    }
    want = {case + (m,): expect for case, expect in whole.items() for m in (0, 1)}
    want.update({case + (m,): expect[m] for case, expect in shared.items() for m in (0, 1)})
    src, exe = tmp_path / "rule.hip", tmp_path / "rule"
    src.write_text(DRIVER)
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    asked = "\n".join(" ".join(str(v) for v in case) for case in want)
    got = subprocess.run([str(exe)], input=asked, capture_output=True, text=True, timeout=60).stdout.split("\n")
    for (case, expect), line in zip(want.items(), got):
        assert tuple(int(v) for v in line.split()) == expect, case


def sides(bytes_an_element):
    """Element counts around every limit, of whole and of shared lines."""
    out = []
    if bytes_an_element > 100:
        out = [1 << 21, (1 << 21) + 32]
    elif bytes_an_element < 28:
        out = [(1 << 21) - 32, 1 << 21]
    for limit, step in ((16 * MIB, 1), (56 * MIB, 32), (264 * MIB, 32), (264 * MIB, 1)):
        n = limit // bytes_an_element
        if step == 32:
            n -= n % 32
            out += [n, n + 32]
        else:
            n -= 1 - n % 2
            out += [n, n + 2]
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("setting,record,message", [((64, 18, 13), 124, 96), ((64, 9, 13), 44, 32), ((64, 3, 13), 12, 8)])
def test_both_sides_match_the_fused_call(setting, record, message):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_04909_amd import bicop as B
    prm, sd = B.Params(*setting), B.Seeds(11, 12, 13, 14)
    assert B.rand_bytes(B.BC_OP_DRELU, prm, 1 << 20) == record << 20 and 8 * B.msg_words(prm.npos) == message
    for calls, counts in (("records", sides(record)), ("messages", sides(message))):
        for n in counts:
            gen = torch.Generator(device="cuda").manual_seed(n)
            x0, x1 = (torch.randint(-(1 << 62), 1 << 62, (n,), generator=gen, device="cuda") for _ in range(2))
            want = B.drelu(x0, x1, prm, sd)
            if calls == "records":
                got = B.drelu_pre(x0, x1, prm, B.rand_expand(B.BC_OP_DRELU, prm, sd, n))
            else:
                d = B.drelu_reply(B.drelu_send(0, x0, prm, sd), B.drelu_send(1, x1, prm, sd), prm, sd)
                got = tuple(B.drelu_finish(p, d[p], prm, sd) for p in (0, 1))
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), (calls, n)
