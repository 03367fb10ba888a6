"""Host rules compiled with g++ from paper_2601_16294_amd/csrc/sfc_model.cpp and its
headers: ``build`` takes the body of a loop over calls read from stdin and returns a
function from calls (tuples of numbers) to the tuples of integers they print."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = f"{ROOT}/paper_2601_16294_amd/csrc"
MAIN = '''
#include <stdio.h>
#include "sfc_model.h"
#include "sfc_params.h"
#include "sfc_validate.h"
int main() {
  %s
  return 0;
}
'''


def build(directory, body):
    src, exe = os.path.join(directory, "rule.cpp"), os.path.join(directory, "rule")
    with open(src, "w") as f:
        f.write(MAIN % body)
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{ROOT}/include",
                    f"-I{CSRC}", src, f"{CSRC}/sfc_model.cpp", "-o", exe], check=True)

    def run(calls):
        text = "\n".join(" ".join(str(v) for v in c) for c in calls)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        return [tuple(int(x) for x in line.split()) for line in out if line]
    return run
