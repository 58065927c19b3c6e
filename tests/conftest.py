import collections
import ctypes
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def _gpu_present():
    try:
        import torch
        return torch.cuda.is_available()
    except Exception:
        return False


def pytest_collection_modifyitems(config, items):
    if _gpu_present():
        return
    skip = pytest.mark.skip(reason="no GPU in this container")
    for item in items:
        if "gpu" in item.keywords:
            item.add_marker(skip)


Route = collections.namedtuple("Route", "kernels fold nsplit rows columns workspace blocks chunks together two_part pair")


@pytest.fixture(scope="session")
def planner(tmp_path_factory):
    """tests/plan_query.cpp, built."""
    so = str(tmp_path_factory.mktemp("plan") / "plan_query.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(ROOT, "tests", "plan_query.cpp")],
                   check=True)
    return ctypes.CDLL(so)


@pytest.fixture(scope="session")
def route(planner):
    """route(op, N, C, H, W, K, R, stride, pad, groups=1, dtype=0, workspace=None, S=None): what the planner does with such a
    pass (and a workspace of so many bytes; filters R x S, or R x R), so that a test written for one set of kernels ("fp32",
    "split", "direct" or "window") can assert that it reaches them.  Of the window kernel also the channel blocks per step and
    the chunks; together: a grouped bf16 backward-filter in one launch of each kernel; two_part: a split pass that runs on two
    half-precision parts where its operands' range lets it; pair: one on four-wave tiles."""
    query = planner.plan_query

    def ask(op, N, C, H, W, K, R, stride, pad, groups=1, dtype=0, workspace=None, S=None):
        out = (ctypes.c_longlong * 11)()
        assert query(op, N, C, H, W, K, R, R if S is None else S, stride, pad, groups, dtype,
                     ctypes.c_longlong(-1 if workspace is None else workspace), out) == 0
        return Route(("fp32", "split", "direct", "window")[out[0]], *list(out)[1:])
    return ask


# Normalised max errors the parity tests measured, printed once at the end of the run (also under -q).
_PARITY = []


@pytest.fixture
def parity_record():
    def record(tag, err, tol):
        _PARITY.append((tag, float(err), float(tol)))
    return record


def pytest_terminal_summary(terminalreporter):
    if not _PARITY:
        return
    terminalreporter.write_line("normalised max error vs the CPU oracle (whole tensors):")
    for tag, err, tol in _PARITY:
        terminalreporter.write_line("  %-44s %.3e  (bar %.1e)" % (tag, err, tol))
