"""The race-hunting build (a workgroup fence after every phase of the forward and every tile or step of the
backward kernels) against the release build: same arithmetic in the same order, so every output must agree
bit for bit.  A difference would mean the release build reads a tile buffer that is being refilled, or the
other way round.

Every case runs twice, plainly and with profile records, which keep the queues and a launch for each kernel; and it says
what the plain call launches (test_launch_rules_host.py checks that, and that no kernel of any head size is left out)."""
import os
import subprocess
import sys
import tempfile

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# (lengths, Hq, Hkv, d_qk, d_v, forward, backward): several tiles per sample and ragged tails, every workgroup shape and
# head size, items handed over from queues (more of them than workgroups fit on the chip), the wrapped block order of long
# samples, partial sums of head parts
LONG = [9000, 5197, 1300, 700, 257, 129, 31, 26]  # 16640 tokens
CASES = [
    # one launch for dK/dV and dQ; few rounds of the forward
    ([512, 256, 128, 64, 64], 4, 4, 64, 64, "halves", "one launch interleaved"),
    ([1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 200, 257, 5, 269], 4, 1, 128, 128, "singles", "one launch interleaved"),
    ([700, 129, 256, 257, 31, 1, 400], 3, 3, 128, 128, "halves", "one launch interleaved"),
    ([900, 333, 1], 2, 2, 192, 128, "halves", "one launch"),
    ([5197, 300], 8, 8, 64, 64, "halves", "one launch interleaved"),
    ([3000, 700, 130], 16, 4, 128, 128, "singles", "one launch"),
    ([700, 129, 1], 16, 8, 64, 64, "singles", "one launch"),
    ([700, 129, 1], 16, 8, 192, 128, "singles", "four waves"),
    ([100, 128, 129, 60, 31, 33, 257, 90] * 4, 32, 8, 128, 128, "pairs", "one launch"),
    ([2400, 1100, 596], 12, 12, 128, 128, "256-row tiles", "one launch interleaved"),
    ([97, 64, 33, 129] * 3, 8, 8, 64, 64, "256-row tiles", "one launch interleaved"),
    ([4000, 3000, 2500, 1500, 1000, 288], 12, 4, 192, 128, "256-row tiles", "four waves"),
    # queues and two launches
    (LONG, 16, 8, 64, 64, "pairs queued", "eight waves"),
    (LONG, 16, 8, 128, 128, "pairs queued", "eight waves"),
    (LONG, 16, 8, 192, 128, "pairs queued", "four waves"),
    (LONG, 24, 24, 64, 64, "256-row tiles queued", "eight waves"),
    (LONG, 10, 10, 192, 128, "256-row tiles queued", "four waves"),
    ([400] * 20 + [700, 513, 257, 330, 200], 24, 24, 128, 128, "256-row tiles queued", "four waves"),
    ([30] * 170, 16, 8, 64, 64, "singles", "four waves"),
    (LONG + [10000, 300], 8, 1, 128, 128, "pairs queued", "eight waves"),  # eight parts: partial sums
    ([700, 257, 40], 72, 8, 128, 128, "halves", "eight waves"),
]

RUNNER = r"""
import hashlib, json, sys
sys.path.insert(0, %(root)r)
import torch
from paper_2503_07680_amd.runner import PackedAttention
import paper_2503_07680_amd as H
out = {}
def run(key, pa, ins, profile):
    for x in (pa.o, pa.dq, pa.dk, pa.dv):
        x.fill_(float("nan"))
    pa.forward(*ins[:3], profile=profile)
    pa.backward(*ins, profile=profile)
    torch.cuda.synchronize()
    for name in ("o", "lse", "dq", "dk", "dv"):
        x = getattr(pa, name)
        assert not torch.isnan(x).any(), (key, name)
        out["%%s %%s" %% (key, name)] = hashlib.sha256(x.contiguous().view(torch.uint8).cpu().numpy().tobytes()).hexdigest()
for i, (lengths, Hq, Hkv, d, e) in enumerate(%(cases)r):
    for rows in (None, 128) if Hq // Hkv %% 2 else (None,):   # odd groups: 128-row query tiles too
        pa = PackedAttention(lengths, sum(lengths), Hq, Hkv, d, e, with_profile=True, fwd_tile_rows=rows)
        gen = torch.Generator(device=pa.device).manual_seed(80 + i)
        ins = [pa.buffer(h, w).normal_(generator=gen) for h, w in ((Hq, d), (Hkv, d), (Hkv, e), (Hq, e))]
        pa.alloc_backward()
        for profile in (False, True):
            run("case %%d rows %%s records %%s" %% (i, rows, profile), pa, ins, profile)
        del pa, ins
    print("case", i, "done with", H.library_path(), flush=True)
json.dump(out, open(sys.argv[1], "w"))
"""


def run_with(library, path):
    import json
    env = dict(os.environ)
    if library:
        env["HBP_LIBRARY"] = library
    else:
        env.pop("HBP_LIBRARY", None)
    code = RUNNER % {"root": ROOT, "cases": [c[:5] for c in CASES]}
    r = subprocess.run([sys.executable, "-c", code, path], env=env, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                       text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-3000:]
    assert ("libhbp_racehunt.so" in r.stdout) == bool(library), r.stdout[-500:]
    with open(path) as f:
        return json.load(f)


def test_release_and_race_hunting_builds_agree_bit_for_bit():
    from paper_2503_07680_amd import build as B
    assert os.path.exists(B.LIB_RACE_HUNT), "build the library first (python -m paper_2503_07680_amd.build)"
    odd = sum((c[1] // c[2]) % 2 for c in CASES)
    with tempfile.TemporaryDirectory() as tmp:
        release = run_with(None, os.path.join(tmp, "release.json"))
        fenced = run_with("libhbp_racehunt.so", os.path.join(tmp, "fenced.json"))
        assert len(release) == 10 * (len(CASES) + odd)
        assert release == fenced, [k for k in release if release[k] != fenced.get(k)]
