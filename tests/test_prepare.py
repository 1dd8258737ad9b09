"""moe_prepare raises every LDS limit: each call that raises one sits in a prepare_ function, and every
prepare_ function of a source file is called by moe_prepare (no GPU; read from the sources)."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2006_16668_amd", "csrc")


def _read(name):
    with open(os.path.join(CSRC, name)) as f:
        return f.read()


def test_every_limit_is_raised_by_a_prepare_function():
    # a function starts in column 0; what follows, up to the next one, is its body
    head = re.compile(r"^(?:static |inline )*int (\w+)\([^;{]*\{", re.M)
    calls = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip"))):
        text = _read(os.path.basename(path))
        for m in re.finditer(r"ensure_lds_limit\(", text):
            name = [h.group(1) for h in head.finditer(text, 0, m.start())][-1]
            assert name.startswith("prepare_"), (os.path.basename(path), name)
            calls += 1
    assert calls >= 6


def test_moe_prepare_calls_every_prepare_function():
    declared = set(re.findall(r"^int (prepare_\w+)\(\);", _read("common.h"), re.M))
    body = re.search(r"^int moe_prepare\(void\) \{(.*?)^\}", _read("api.hip"), re.M | re.S).group(1)
    assert declared and declared == set(re.findall(r"moe::(prepare_\w+)\(\)", body))
    for path in glob.glob(os.path.join(CSRC, "*.hip")):      # and every template of one is listed by its file's
        text = _read(os.path.basename(path))
        for name in re.findall(r"^(?:static )?int (prepare_\w+)\(\) \{", text, re.M):
            if name not in declared:
                owners = [re.search(r"^int %s\(\) \{.*?^\}" % d, text, re.M | re.S) for d in declared]
                assert any(o and (name + "<") in o.group(0) for o in owners), name
