"""The publisher's chunks are stored written through: a flag may follow only once every wave's stores have left it.  Read from the
assembly that the compiler makes of the library's own source, so no GPU is needed and no unordered store has to be caught in the act."""
import re
import subprocess

from paper_2605_02953_amd import build


def _kernel(source, name, tmp_path):
    """Instructions of kernel `name`, labels left out."""
    out = tmp_path / "kernel.s"
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.run([build.HIPCC] + flags + ["-I", f"{build.HERE}/../include", "--cuda-device-only", "-S",
                                            f"{build.HERE}/csrc/{source}", "-o", str(out)], check=True, capture_output=True)
    body = re.search(rf"^\w*{name}\w*:.*?^\s*s_endpgm", out.read_text(), re.S | re.M).group(0)
    return [line.split(";")[0].strip() for line in body.splitlines() if re.match(r"\s+[a-z]", line)]


def test_published_chunks_leave_every_wave_before_the_flag(tmp_path):
    code = _kernel("api.hip", "publish_chunks_kernel", tmp_path)
    stores = [i for i, ins in enumerate(code) if ins.startswith("buffer_store")]
    assert stores and all("sc0" in code[i] and "sc1" in code[i] for i in stores)
    # from the last of a round's stores on: the wait for all of them, then the barrier, then the flag
    after = code[stores[-1] + 1:]
    barrier = next(i for i, ins in enumerate(after) if ins.startswith("s_barrier"))
    assert any(re.match(r"s_waitcnt.*vmcnt\(0\)", ins) for ins in after[:barrier]), after[:barrier + 1]
    # and the flag itself needs no write-back of the cache
    assert not any(ins.startswith("buffer_wbl2") for ins in code)
