"""The rules that pick a mesh's tiles, on the CPU: compiled for the host from the
header the library uses.  The tile kernels form a lane's offset from its tile in
32 bits; a configuration in which it would wrap is never picked."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_tiles_address_the_mesh(tmp_path):
    exe = str(tmp_path / "check_tiles")
    subprocess.check_call(["/opt/rocm/bin/hipcc", "-O1", "-std=c++17", "--offload-arch=gfx950",
                           os.path.join(HERE, "host", "check_tiles.hip"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(out.stdout)
    assert out.returncode == 0, out.stdout
    assert " 0 failures" in out.stdout
