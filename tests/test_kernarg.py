"""Where the walk kernels take the address of their arguments.  The builtin that
gives it is null in a function that is called, so it may stand in kernels alone:
looked for in code compiled without inlining, where every function that is not
forced into its caller stays one."""
import os
import re
import subprocess

from paper_2511_20317_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_argument_segment_is_taken_in_kernels_alone(tmp_path):
    out = str(tmp_path / "kernarg.ll")
    subprocess.run([build.HIPCC] + build.HIP_FLAGS +
                   ["-O1", "-Xclang", "-fno-inline", "--cuda-device-only", "-S", "-emit-llvm",
                    os.path.join(HERE, "kernarg_shim.hip"), "-o", out],
                   check=True, capture_output=True)
    kernels, called, function = 0, [], None
    with open(out) as f:
        for line in f:
            if line.startswith("define"):
                function = line
            elif line.startswith("}"):
                function = None
            elif function and "kernarg.segment.ptr" in line:
                if "amdgpu_kernel" in function:
                    kernels += 1
                else:
                    called.append(re.search(r"@(\S+?)\(", function).group(1))
    assert kernels >= 2          # both kernels of the shim
    assert not called, called
