"""Every test that is written down runs: no module of this folder defines a name
twice at its top level (the later definition would replace the earlier one, and
pytest would never see it)."""
import ast
import glob
import os

HERE = os.path.dirname(os.path.abspath(__file__))


def test_no_name_is_defined_twice():
    twice = []
    for path in sorted(glob.glob(os.path.join(HERE, "*.py"))):
        seen = set()
        for node in ast.parse(open(path).read()).body:
            if isinstance(node, (ast.FunctionDef, ast.ClassDef)):
                if node.name in seen:
                    twice.append(f"{os.path.basename(path)}:{node.lineno} {node.name}")
                seen.add(node.name)
    assert not twice, twice
