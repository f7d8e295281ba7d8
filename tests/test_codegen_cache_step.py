"""The cache step's bucket atomic is in flight during the access and retention
that follow it: in the assembly that hipcc makes of cache.hip, no variant of the
kernel waits for it (a wait for every outstanding memory operation) in the next
instructions.  A 64-bit use of the returned position has put such a wait right
behind the atomic."""
import re
import subprocess

from paper_2609_04895_amd import build


def test_no_wait_behind_the_bucket_atomic(tmp_path):
    out = tmp_path / "cache.s"
    src = build.os.path.join(build._HERE, "csrc", "cache.hip")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.check_call([build.HIPCC, *flags, "--offload-device-only", "-S", src, "-o", str(out)])
    kernel, since, seen = None, None, {}
    for line in out.read_text().splitlines():
        m = re.match(r"(_ZN\S*cache_step_kernel\S*):", line)
        if m:
            kernel, since = m.group(1), None
        elif re.match(r"\.Lfunc_end", line):
            kernel = None
        if kernel is None:
            continue
        ins = line.strip()
        if ins.startswith("global_atomic_add ") and "sc0" in ins:
            assert kernel not in seen, kernel
            since = seen[kernel] = 0
        elif since is not None and ins and ins[0] not in ".;":
            if "s_waitcnt" in ins and "vmcnt(0)" in ins:
                since = None
            else:
                since += 1
                seen[kernel] = since
    assert len(seen) == 45, len(seen)  # every variant of the kernel
    # what follows up to the first wait is the access (about 80 instructions up)
    assert min(seen.values()) >= 60, min(seen.items(), key=lambda kv: kv[1])
