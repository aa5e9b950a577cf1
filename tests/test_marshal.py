"""The short calls' native marshalling takes plain device tensors only; everything else goes the general way, which converts it or
words its error.  Both ways make the same call."""
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest
import torch

import paper_2509_15148_amd as A
from paper_2509_15148_amd import binding as B
from synth import lognormal_scores
from util import announce, dev


def test_what_is_not_plain_is_left_to_the_general_way():
    m, other = B._marshal, B._marshal.OTHER
    assert m.__file__.endswith("_marshal.so")                     # the native one
    host, off = torch.zeros(4), torch.zeros(2, dtype=torch.int64)
    assert other not in (A.OK, A.ERR_INVALID_ARG, A.ERR_SHAPE, A.ERR_WORKSPACE, A.ERR_CAPACITY, A.ERR_HIP)
    for handle in (None, 0, "x", 1.5):
        assert m.calibrate_online(handle, host) == other
    assert m.calibrate_online(1 << 20, host) == other and m.calibrate_online(1 << 20, [1.0]) == other and m.calibrate_online(1 << 20) == other
    for alphas in ([0.1], (0.1,), [], [1], np.array([0.1]), "ab", [0.1] * 9):
        assert m.classify_ordinal(1 << 20, host, alphas, None, None, host.to(torch.uint8), None) == other
        assert m.classify_conditional(host, off, host, off, alphas, host.int(), None, host.to(torch.uint8)) == other
    fake = torch.empty(4, device="meta")
    assert m.calibrate_online(1 << 20, fake) == other


@pytest.mark.parametrize("native", ["absent", "not loadable"])
def test_import_without_the_native_module(tmp_path, native):
    """libatts.so is all that the package needs: the short calls then take the general way, with its wording of errors."""
    where = os.path.dirname(B.__file__)
    shutil.copytree(where, tmp_path / "paper_2509_15148_amd", ignore=shutil.ignore_patterns("_marshal.so", "_build", "csrc", "__pycache__"))
    if native == "not loadable":
        (tmp_path / "paper_2509_15148_amd" / "_marshal.so").write_bytes(b"no library")
    code = ("import torch, paper_2509_15148_amd as A\nassert A.__file__.startswith(%r), A.__file__\nprint(A.atts_classic_workspace_bytes(100))\n"
            "c = A.Calib.__new__(A.Calib); c.handle = A.binding.ctypes.c_void_p()\n"
            "for call in (lambda: A.atts_calibrate_online(c, torch.zeros(4)), lambda: A.atts_classify_ordinal(c, torch.zeros(4), [0.1], None, None, "
            "torch.zeros(4, dtype=torch.uint8), None)):\n"
            "    try: call()\n    except A.AttsError as e: assert 'device tensor' in str(e), e\n    else: raise AssertionError\n" % str(tmp_path))
    r = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True, env={**os.environ, "PYTHONPATH": str(tmp_path)})
    assert r.returncode == 0 and int(r.stdout) == A.atts_classic_workspace_bytes(100), r.stderr


@pytest.mark.parametrize("bad", ["x", None, [1]])
def test_numbers_of_a_wrong_type(bad, monkeypatch):
    """A TypeError, whose message says what is wrong, from every entry that takes numbers from its caller."""
    monkeypatch.setattr(B, "_ptr", lambda *args: None)             # host tensors get as far as the numbers
    monkeypatch.setattr(B, "_stream", lambda: 0)

    class Handle:
        handle = None
    ids, out, x, space = torch.zeros(2, 3, dtype=torch.int32), torch.zeros(2, 4, dtype=torch.int32), torch.zeros(2), torch.zeros(256, dtype=torch.uint8)
    u = torch.zeros(2, 4)
    for call in (lambda: A.Calib(bad), lambda: A.Prefix(Handle, bad), lambda: A.atts_score_drafts(Handle, ids[0], ids, None, bad, None, x, space),
                 lambda: A.atts_score_drafts_cached(Handle, ids, None, bad, None, x, space), lambda: A.atts_prefix_extend_workspace_bytes(Handle, bad),
                 lambda: A.atts_continue_workspace_bytes(Handle, 1, bad, 1), lambda: A.atts_continue_greedy(Handle, ids, out, space, eos_id=bad),
                 lambda: A.atts_continue_sample(Handle, ids, bad, u, out, space), lambda: A.atts_classic_workspace_bytes(bad),
                 lambda: A.atts_classic_threshold(x, bad, x[:1], space), lambda: A.atts_profile_read(bad)):
        with pytest.raises(TypeError, match="interpreted as an integer|must be real number"):
            call()


@pytest.mark.gpu
def test_both_ways_make_the_same_call():
    announce("marshal both ways")
    cal, x = dev(lognormal_scores(500, seed=3)), dev(lognormal_scores(40, seed=4))
    out = {}
    for way in ("native", "general"):
        alphas = [0.05, 0.2] if way == "native" else np.array([0.05, 0.2])
        c = A.Calib(1000)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):                             # on the caller's stream: the scores are written there just before
            y = (cal * 2.0).mul_(0.5)
            r, p, k, t = (torch.empty(n, dtype=d, device="cuda") for n, d in ((40, torch.int32), (40, torch.float32), (40, torch.uint8), (2, torch.float32)))
            A.atts_calibrate_online(c, y)
            A.atts_classify_ordinal(c, x, alphas, r, p, k, t)
            off, xo = dev(np.array([0, 200, 500])), dev(np.array([0, 15, 40]))
            r2, p2, k2 = torch.empty_like(r), torch.empty_like(p), torch.empty_like(k)
            A.atts_classify_conditional(y, off, x, xo, alphas, r2, p2, k2)
        torch.cuda.synchronize()
        out[way] = [v.cpu() for v in (r, p, k, t, r2, p2, k2)]
        c.close()
    assert all(torch.equal(a, b) for a, b in zip(out["native"], out["general"]))


@pytest.mark.gpu
def test_errors_are_worded_as_before():
    announce("marshal errors")
    c, f = A.Calib(64), A.Calib(64)                               # an empty set and a filled one
    x = dev(lognormal_scores(32, seed=5))
    A.atts_calibrate_online(f, x)
    r, k = torch.empty(32, dtype=torch.int32, device="cuda"), torch.empty(32, dtype=torch.uint8, device="cuda")
    for call, text in ((lambda: A.atts_calibrate_online(c, x[::2]), "contiguous"), (lambda: A.atts_calibrate_online(c, x.double()), "dtype"),
                       (lambda: A.atts_calibrate_online(c, x.cpu()), "device tensor"),
                       (lambda: A.atts_calibrate_online(c, torch.cat([x, x, x])), "capacity"),
                       (lambda: A.atts_classify_ordinal(c, x, [0.1], r, None, k, None), "empty"),
                       (lambda: A.atts_classify_ordinal(c, x, [0.1], r[:5], None, k, None), "M elements"),
                       (lambda: A.atts_classify_ordinal(f, x, [0.1], None, x, k, None), "without ranks"),
                       (lambda: A.atts_classify_ordinal(c, x, [0.1], r, None, k, x), "n_alpha"),
                       (lambda: A.atts_classify_ordinal(c, x, [1.5], r, None, k, None), "inside (0, 1)")):
        with pytest.raises(A.AttsError) as e:
            call()
        assert e.value.code in (A.ERR_INVALID_ARG, A.ERR_CAPACITY) and text in str(e.value), text
    c.close()
    f.close()
    with pytest.raises(A.AttsError):                              # a closed handle
        A.atts_calibrate_online(c, x)
