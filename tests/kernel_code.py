"""Instructions of the kernels built into libtpo.so, from the disassembly of its own code objects; no GPU needed."""
import os
import re
import subprocess
import tempfile

from kernel_metadata import _code_objects
from paper_2604_19906_amd import tpo

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")


def instructions():
    """Mangled kernel name -> its instructions, in order."""
    found = {}
    with open(tpo.LIB_PATH, "rb") as f:
        blob = f.read()
    for elf in _code_objects(blob):
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(elf)
            f.flush()
            text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", f.name],
                                  capture_output=True, text=True, check=True).stdout
        code = None
        for line in text.split("\n"):
            m = re.match(r"(?:[0-9a-f]+ )?<(\w+)>:", line)
            if m:
                code = found.setdefault(m.group(1), [])
            elif code is not None and line.strip():
                code.append(line.split("//")[0].strip())
    return found
