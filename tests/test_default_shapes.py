"""What a program gets that loads no launch table: the shapes of the shipped one."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_defaults_are_the_shipped_two_sweep_and_restriction_shapes():
    code = (
        "import json, os, sys; sys.path.insert(0, %r)\n"
        "from paper_1201_3185_amd import qumond as Q\n"
        "table = json.load(open(os.path.join(os.path.dirname(Q.__file__), 'launch_shapes_mi355x.json')))['smoother']\n"
        "seen = 0\n"
        "for e in table:\n"
        "    n, fp = e['n'], bool(e['fp32'])\n"
        "    if e.get('fused') == 1:\n"
        "        assert Q.tune_get_fused(n, fp) == (e['variant'], e['kchunk']), (e, Q.tune_get_fused(n, fp))\n"
        "        seen += 1\n"
        "    if 'rr' in e:\n"
        "        assert Q.tune_get_rr(n, fp) == e['rr'], (e, Q.tune_get_rr(n, fp))\n"
        "        seen += 1\n"
        "assert seen == 20\n"
        "for fp in (False, True):\n"      # 1025^3, which no table holds, as 513^3
        "    assert Q.tune_get_fused(1025, fp) == Q.tune_get_fused(513, fp) == (8, 0)\n"
        "    assert Q.tune_get_rr(1025, fp) == Q.tune_get_rr(513, fp) == 7\n"
        "print('ok')\n" % ROOT)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
