"""A second function of the same name in a file takes the first one's place, and its cases no longer run."""
import ast
import collections
import glob
import os

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.parametrize("path", sorted(os.path.basename(p) for p in glob.glob(os.path.join(HERE, "*.py"))))
def test_no_function_is_defined_twice(path):
    with open(os.path.join(HERE, path)) as f:
        names = collections.Counter(n.name for n in ast.parse(f.read()).body if isinstance(n, ast.FunctionDef))
    assert [n for n, count in names.items() if count > 1] == []
