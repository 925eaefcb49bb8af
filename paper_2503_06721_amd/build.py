"""Build libwdirac.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2503_06721_amd.build          # or build() from Python

Every HIP source is compiled to an object under _build/ (in parallel; the
hop sources, whose kernels are many, in parts), then linked into paper_2503_06721_amd/libwdirac.so next to this file.
"""
import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, 'csrc')
BUILD = os.path.join(HERE, '_build')
LIB = os.path.join(HERE, 'libwdirac.so')
SOURCES = ['api.hip', 'rep.hip', 'blas.hip', 'force.hip', 'stream.hip', 'clover.hip', 'hmc.hip',
           'cg_tiny.hip', 'hop_clover.hip']
# (source, WD_PART): each part holds the kernels of some precisions, projectors
# and representation dimensions (the longest first)
PARTS = [('hop.hip', k) for k in range(8)] + [('hop_mr.hip', k) for k in range(4)]
HIPCC = os.environ.get('HIPCC', '/opt/rocm/bin/hipcc')
ARCH = 'gfx950'
FLAGS = [
    '-O3', '-std=c++17', '-fPIC', f'--offload-arch={ARCH}',
    # packed FP32 instructions are kept out of the generated code
    '-Xclang', '-target-feature', '-Xclang', '-packed-fp32-ops',
    '-Wno-unused-command-line-argument',
]


def _compile(job):
    src, part = job
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ('' if part is None else f'_{part}') + '.o')
    define = [] if part is None else [f'-DWD_PART={part}']
    cmd = [HIPCC, *FLAGS, *define, '-I', CSRC, '-c', os.path.join(CSRC, src), '-o', obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f'hipcc failed on {src}:\n{" ".join(cmd)}\n{res.stdout}\n{res.stderr}')
    return obj


def build(verbose=False, jobs=None):
    """Compile every HIP source for gfx950 and link libwdirac.so.  Always rebuilds."""
    os.makedirs(BUILD, exist_ok=True)
    work = PARTS + [(src, None) for src in SOURCES]
    jobs = jobs or min(len(work), max(1, (os.cpu_count() or 2)))
    with concurrent.futures.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, work))
    tmp = LIB + '.tmp'
    cmd = [HIPCC, '-shared', '-fPIC', f'--offload-arch={ARCH}', *objs, '-o', tmp]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f'link failed:\n{" ".join(cmd)}\n{res.stdout}\n{res.stderr}')
    os.replace(tmp, LIB)
    if verbose:
        print(f'built {LIB}')
    return LIB


if __name__ == '__main__':
    build(verbose=True)
    sys.exit(0)
