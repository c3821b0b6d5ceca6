"""The HIP path and the oracle share no code, and the benchmark refuses more than one GPU.
No GPU needed."""
import os
import re
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _sources(folder, exts):
    out = []
    for base, _, files in os.walk(os.path.join(ROOT, folder)):
        if "__pycache__" in base:
            continue
        out += [os.path.join(base, f) for f in files if f.endswith(exts)]
    return out


def test_product_path_never_touches_the_oracle():
    files = _sources("paper_2505_04421_amd", (".py", ".h", ".hip")) + _sources("include", (".h",))
    assert files
    for path in files:
        text = open(path).read()
        assert not re.search(r"\boracle\b", text), path + " mentions the oracle"


def test_oracle_is_independent_of_the_hip_path():
    files = _sources("oracle", (".py", ".c", ".h"))
    assert files
    for path in files:
        text = open(path).read()
        assert "paper_2505_04421_amd" not in text and "liblonger" not in text and "ctypes" not in text, path


def _arguments(text, start):
    """The top-level arguments of the call whose opening parenthesis is at text[start]."""
    depth, args, last = 0, [], start + 1
    for i in range(start, len(text)):
        c = text[i]
        if c in "([{":
            depth += 1
        elif c in ")]}":
            depth -= 1
            if depth == 0:
                return args + [text[last:i].strip()]
        elif c == "," and depth == 1:
            args.append(text[last:i].strip())
            last = i + 1
    raise AssertionError("unbalanced call")


def test_buffer_stores_take_no_scalar_offset():
    """A 16-byte buffer store reads its data for two more cycles after its issue, and the compiler does not keep the registers for that
    long behind a store whose offset is in a scalar register: pieces of results were replaced now and then.  So the scalar offset of
    every buffer store in the sources is the literal 0, and no inline assembly stores through a buffer."""
    calls = 0
    for path in _sources("paper_2505_04421_amd", (".h", ".hip")):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"__builtin_amdgcn_(raw|struct)\w*buffer_store\w*\s*(?=\()", text):
            args = _arguments(text, m.end())
            assert args[4 if m.group(1) == "struct" else 3] == "0", "%s: %s%s" % (path, m.group(0), args)
            calls += 1
        assert "buffer_store_" not in re.sub(r"__builtin_amdgcn_\w+", "", text), path
    assert calls


def test_input_generator_holds_no_model_arithmetic():
    text = open(os.path.join(ROOT, "longer_synth", "__init__.py")).read()
    for word in ("softmax", "layer_norm", "erf(", "import torch", "paper_2505_04421_amd", "from oracle"):
        assert word not in text, word


def test_bench_refuses_more_than_one_gpu():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 2 and "ONE GPU" in r.stderr and r.stdout.strip() == ""


def test_benchmark_touches_the_oracle_only_in_its_cpu_baseline_leg():
    text = open(os.path.join(ROOT, "bench.py")).read()
    imports = [m.start() for m in re.finditer(r"from oracle import|import oracle", text)]
    assert len(imports) == 1
    leg = text.index("def cpu_oracle_leg(")
    nxt = text.index("\ndef ", leg + 1)
    assert leg < imports[0] < nxt
    assert "orc." not in text[:leg] and "orc." not in text[nxt:]
