"""What a call hands to the runtime, without a GPU: builds launch_probe.cpp, whose own launch functions stand in for the runtime's, and
drives it over a pipe."""
import atexit
import collections
import functools
import os
import subprocess
import tempfile

import paper_1805_00907_amd as glowmi

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.dirname(os.path.abspath(glowmi.__file__))

Launch = collections.namedtuple("Launch", "kernel lds limit")


@functools.lru_cache(maxsize=None)
def _built(library):
    tmp = tempfile.TemporaryDirectory()
    atexit.register(tmp.cleanup)
    exe = os.path.join(tmp.name, "launch_probe")
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-D__HIP_PLATFORM_AMD__=1", "-isystem", "/opt/rocm/include", "-o", exe,
                    os.path.join(HERE, "launch_probe.cpp"), library, f"-Wl,-rpath,{os.path.dirname(library)}", "-L/opt/rocm/lib",
                    "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"], check=True, capture_output=True)
    return exe


class LaunchProbe:
    """A process of its own: nothing has been launched in it yet."""

    def __init__(self, library=None):
        self.process = subprocess.Popen([_built(library or os.path.join(PKG, "libglowmi.so"))], stdin=subprocess.PIPE,
                                        stdout=subprocess.PIPE, text=True)

    def _ask(self, line):
        self.process.stdin.write(line + "\n")
        self.process.stdin.flush()
        return self.process.stdout.readline().strip()

    def knob(self, name, value):
        assert self._ask(f"knob {name} {value}") == "ok", name

    def reset(self):
        assert self._ask("reset") == "ok"

    variant = ""                                             # the last call's

    def sequence(self, x_shape, layers, quantized=True, add=()):
        """layers: (output channels, filter size) each; add: which add the sequence input.  The launches of one call."""
        bits = sum(1 << i for i in add)
        said = self._ask(f"seq {int(quantized)} {len(layers)} {bits} {' '.join(map(str, x_shape))} " + " ".join(f"{k} {r}" for k, r in layers)).split()
        assert said[0] == "0", said
        self.variant = said[1]
        return [Launch(k, int(lds), int(limit)) for k, lds, limit in (s.rsplit("|", 2) for s in said[2:])]

    def versus(self, name, value, repeats=3000):
        """Median nanoseconds of a call like the last one: with that switch, with none."""
        return tuple(map(int, self._ask(f"versus {name} {value} {repeats}").split()))

    def close(self):
        self.process.stdin.close()
        self.process.wait(timeout=30)

    def __enter__(self):
        return self

    def __exit__(self, *_):
        self.close()
