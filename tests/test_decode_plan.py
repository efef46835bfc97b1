"""The launch plan of a decode (csrc/plan.hpp, host code), compiled here on its own and looked at
directly: what it may never do, and the lines of its rules."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_03458_amd", "csrc")
FIELDS = ("n_chunk", "g_chunk", "n_wg", "group", "order", "ws_parts")
MAIN = """
#include <cstdio>
#include "plan.hpp"
int main() {
    int a[8];
    while (scanf("%d %d %d %d %d %d %d %d", a, a + 1, a + 2, a + 3, a + 4, a + 5, a + 6, a + 7) == 8) {
        const kvarn::DecodePlan p = kvarn::plan_decode(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7]);
        printf("FORMAT\\n", ARGS);
    }
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """plans([(batch, n_kv, n_q, bits, max_len, n_sink, max_blocks, equal), ...]) -> list of plan dicts."""
    d = tmp_path_factory.mktemp("plan")
    text = MAIN.replace("FORMAT", " ".join(["%d"] * len(FIELDS))).replace("ARGS", ", ".join("p." + f for f in FIELDS))
    (d / "main.cpp").write_text(text)
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/bin/amdclang++"
    subprocess.check_call([cxx, "-O1", "-std=c++17", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "plan")])

    def run(calls):
        text = "\n".join(" ".join(map(str, c)) for c in calls)
        out = subprocess.run([str(d / "plan")], input=text, capture_output=True, text=True, check=True).stdout
        return [dict(zip(FIELDS, map(int, line.split()))) for line in out.splitlines()]
    return run


def call(streams, tokens, group=4, bits=2, n_kv=8, n_sink=0, equal=0):
    """A call of that many (sequence, kv head) pairs, with room for the tokens."""
    assert streams % n_kv == 0
    return (streams // n_kv, n_kv, n_kv * group, bits, tokens, n_sink, tokens // 128 + 1, equal)


def _random_calls(n):
    rng = random.Random(5)
    out = []
    for _ in range(n):
        n_kv, batch = rng.choice([1, 2, 3, 4, 8, 16]), int(2 ** rng.uniform(0, 11))
        sink, tokens = rng.choice([0, 0, 1, 100, 128, 1024]), int(2 ** rng.uniform(0, 17))
        out.append((batch, n_kv, n_kv * rng.randint(1, 16), rng.choice([2, 4]), tokens, sink,
                    rng.choice([tokens // 128 + 1, tokens // 300]), rng.randint(0, 1)))
    return out


def test_plans_fit_the_card_and_the_workspace(plans):
    """Every plan covers the group's heads, stays within a CU's waves, and writes no more partials than
    the workspace that the library asks for has room for (a caller's buffer of that size is all there is)."""
    from paper_2606_03458_amd import kvarn as K
    lib, calls = K.lib(), _random_calls(20000)
    for c, p in zip(calls, plans(calls)):
        batch, n_kv, n_q, bits, tokens, sink, blocks, equal = c
        g = n_q // n_kv
        assert p["n_chunk"] * p["g_chunk"] >= g > (p["n_chunk"] - 1) * p["g_chunk"] and p["g_chunk"] <= 8, c
        per_cu = 12 if bits == 2 and p["g_chunk"] <= 4 else 8
        assert 1 <= p["group"] <= per_cu, c
        assert p["n_wg"] == 1 or 1 < p["n_wg"] <= min(p["ws_parts"], 32), c
        assert not p["order"] or (batch <= 128 and p["n_wg"] == 1 and not equal), c
        params = K.kvarn_params_init(bits, n_sink=sink)
        cache = K.kvarn_cache(batch, n_kv, blocks)
        ws = lib.kvarn_decode_workspace_bytes(ctypes.byref(params), ctypes.byref(cache), n_q, tokens)
        assert ws == batch * n_q * p["ws_parts"] * 260 * 4, c


@pytest.mark.parametrize("streams,tokens,kw,wg,waves", [
    # equally long (a step): four waves, not the whole CU that ragged sequences take
    (264, 16384, dict(equal=1), 1, 4), (384, 32768, dict(equal=1), 1, 4), (512, 8192, dict(equal=1, group=8), 1, 4),
    # ragged: the whole CU from where the second round of workgroups is worth its while
    (264, 16384, dict(), 1, 4), (352, 32768, dict(), 1, 4), (360, 16384, dict(), 1, 12), (384, 16384, dict(), 1, 12),
    (512, 16384, dict(group=8), 1, 8), (264, 16384, dict(group=8), 1, 8), (264, 12160, dict(bits=4), 1, 4), (512, 8191, dict(), 1, 4), (520, 16384, dict(), 1, 4),
    # below a workgroup per CU: several where a ragged batch would leave CUs idle
    (144, 33000, dict(bits=4), 3, 4), (160, 16384, dict(), 4, 4), (176, 33000, dict(bits=4), 4, 4), (192, 33000, dict(group=8), 4, 4),
    (192, 33000, dict(group=8, equal=1), 1, 8), (176, 33000, dict(equal=1), 1, 12), (176, 8192, dict(), 1, 12), (240, 33000, dict(bits=4), 4, 4), (240, 33000, dict(), 1, 12), (248, 33000, dict(bits=4), 1, 8),
    (96, 33000, dict(group=16, bits=4), 4, 4), (128, 16384, dict(equal=1), 6, 4),
    # more than 768: as many waves as share the longest sequences of a ragged batch
    (832, 16384, dict(n_kv=1), 1, 4), (832, 3000, dict(n_kv=1), 1, 2), (1024, 16384, dict(bits=4), 1, 2),
    (1152, 2048, dict(), 1, 4), (1152, 1920, dict(), 1, 2), (1472, 2048, dict(), 1, 4), (1480, 8192, dict(), 1, 2), (1536, 8192, dict(), 1, 2), (1544, 8192, dict(), 1, 4),
    (1544, 1920, dict(), 1, 1), (1544, 2100, dict(), 1, 4), (1544, 2100, dict(equal=1), 1, 1), (3064, 8192, dict(), 1, 4), (3072, 8192, dict(), 1, 1),
    (1152, 600, dict(bits=4), 1, 4), (1152, 511, dict(bits=4), 1, 1), (1288, 600, dict(bits=4), 1, 1), (2040, 4096, dict(group=8), 1, 4),
    (2048, 4096, dict(group=8), 1, 1), (576, 16384, dict(group=16, bits=4), 1, 4),
])
def test_plan_rules(plans, streams, tokens, kw, wg, waves):
    """Workgroups per stream and waves per workgroup on both sides of each line, for equally long and for
    ragged batches: a plan tuned on one kind made calls of the other up to 1.5 times as long."""
    p, = plans([call(streams, tokens, **kw)])
    assert (p["n_wg"], p["group"]) == (wg, waves)
