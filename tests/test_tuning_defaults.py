"""Every test starts with the library's own choices: the values a fixture sets before each one, and those the tests go back to, are the library's initial ones."""
import ast
import glob
import os
import re

from conftest import ROOT, TUNING_DEFAULTS

CSRC = os.path.join(ROOT, "paper_2605_08151_amd", "csrc")


def _initial():
    api = open(os.path.join(CSRC, "api.hip")).read()
    source = "".join(open(f).read() for f in glob.glob(os.path.join(CSRC, "*.hip")))
    return {key: int(re.search(r"Tunable %s\{(-?\d+)\}" % var, source)[1])
            for key, var in re.findall(r'strcmp\(key, "(\w+)"\) == 0\) \{ specv::(\w+) =', api)}


def test_the_fixture_sets_what_the_library_starts_with():
    assert _initial() == TUNING_DEFAULTS


def test_what_a_test_goes_back_to_is_the_initial_value():
    initial, seen = _initial(), 0
    for path in glob.glob(os.path.join(ROOT, "tests", "test_*.py")):
        for block in ast.walk(ast.parse(open(path).read())):
            for call in (c for s in getattr(block, "finalbody", []) for c in ast.walk(s)):
                if isinstance(call, ast.Call) and getattr(call.func, "attr", "") == "spec_set_tuning" and all(isinstance(a, ast.Constant) for a in call.args):
                    key, value = (a.value for a in call.args)
                    assert value == initial[key], (os.path.basename(path), call.lineno, key, value)
                    seen += 1
    assert seen > 10
