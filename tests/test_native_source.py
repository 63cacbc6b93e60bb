"""What the native fast path of the Python binding has to keep to and no run shows: read from its source."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def source():
    text = open(os.path.join(ROOT, "paper_2506_04985_amd", "csrc", "fptq_native.cpp")).read()
    return re.sub(r"//[^\n]*", "", text)


def bodies(text, head):
    """(start, end) of the braces that follow every match of head, whose last character is the opening one."""
    spans = []
    for m in re.finditer(head, text):
        depth, i = 1, m.end()
        while depth:
            depth += {"{": 1, "}": -1}.get(text[i], 0)
            i += 1
        spans.append((m.end(), i))
    return spans


def test_library_calls_and_allocations_run_without_the_interpreter_lock():
    text = source()
    unlocked = bodies(text, r"\blaunch\(\{[^}]*\}, \[&\] \{") + bodies(text, r"without_gil\(\[&\] \{")
    allocate = bodies(text, r"void allocate\(\)\s*\{")
    inside = lambda m, spans: any(a <= m.start() < b for a, b in spans)
    calls = list(re.finditer(r"\bfptq_\w+\s*\(", text))
    assert len(calls) >= 13 and all(inside(m, unlocked) for m in calls)
    assert all(inside(m, unlocked + allocate) for m in re.finditer(r"\bat::empty\w*\(", text))
    uses = [m for m in re.finditer(r"\ballocate\(\)", text) if not text[:m.start()].endswith("void ")]
    assert len(uses) == 1 and inside(uses[0], unlocked)
    # nothing inside touches Python objects
    assert not any(re.search(r"\bPy[A-Z_]|THPVariable|\btake\(|\bwhere\(|\bcapturing\(", text[a:b]) for a, b in unlocked + allocate)


def test_scratch_comes_from_the_stream_of_the_launch():
    text = source()
    assert re.search(r"const Where w = where\(\);\s*void \*const st = w\.stream;", text)
    assert re.search(r"may_scratch = [^;]*\bxq\.device\(\)\.index\(\) == w\.device;", text)
    assert re.search(r"scratch_bytes = may_scratch \? without_gil\(\[&\] \{ return fptq_linear_scratch_bytes\(M, N, K\); \}\) : 0;", text)
    assert len(re.findall(r"scratch = at::empty\(\{scratch_bytes\}", text)) == 1
