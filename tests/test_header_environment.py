"""include/fdetd.h lists every environment variable that the library reads."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_environment_variable_is_listed():
    csrc = os.path.join(ROOT, "paper_2605_12132_amd", "csrc")
    read = {v for f in os.listdir(csrc) for v in re.findall(r'getenv\("(\w+)"\)', open(os.path.join(csrc, f)).read())}
    text = open(os.path.join(ROOT, "include", "fdetd.h")).read()
    text = text[text.index("/* Environment variables"):text.index("typedef struct")]
    listed = set(re.findall(r"^ \*   (FDETD_\w+)  ", text, re.M))
    assert read and read == listed, (read - listed, listed - read)
