// Host build of the grid searches of the video warm start (chamfer_grid.hip,
// nn_grid.h) under AddressSanitizer; test infrastructure only.  The sources
// compile unchanged against the host stand-in of <hip/hip_runtime.h>; inputs,
// outputs and the workspace are allocations of exactly their size.
//
//   grid_host chamfer DIR       DIR/{s1,s2}.bin -> DIR/{cd,grad2,nn12,nn21}.bin
//   grid_host topk    DIR k3 K  DIR/{s1,sh1,s2}.bin -> DIR/{out_sh,idx}.bin
#include "chamfer.hip"
#include "chamfer_grid.hip"

#include <string>

namespace {

template <class T>
T *filled(uint64_t bytes) {
    void *p = std::malloc(bytes ? bytes : 1);
    std::memset(p, 0xFF, bytes ? bytes : 1);
    return static_cast<T *>(p);
}

float *read_f32(const std::string &path, uint64_t *floats) {
    FILE *f = std::fopen(path.c_str(), "rb");
    if (!f) std::exit(2);
    std::fseek(f, 0, SEEK_END);
    const uint64_t bytes = (uint64_t)std::ftell(f);
    std::fseek(f, 0, SEEK_SET);
    float *p = filled<float>(bytes);
    if (bytes && std::fread(p, 1, bytes, f) != bytes) std::exit(2);
    std::fclose(f);
    *floats = bytes / 4;
    return p;
}

void write_raw(const std::string &path, const void *p, uint64_t bytes) {
    FILE *f = std::fopen(path.c_str(), "wb");
    if (!f || (bytes && std::fwrite(p, 1, bytes, f) != bytes)) std::exit(2);
    std::fclose(f);
}

}  // namespace

int main(int argc, char **argv) {
    if (argc < 3) return 2;
    const std::string mode = argv[1], dir = argv[2];
    uint64_t f1 = 0, f2 = 0, fh = 0;
    float *s1 = read_f32(dir + "/s1.bin", &f1), *s2 = read_f32(dir + "/s2.bin", &f2);
    const uint32_t n1 = (uint32_t)(f1 / 3), n2 = (uint32_t)(f2 / 3);
    if (mode == "chamfer") {
        uint8_t *ws = filled<uint8_t>(dpr::chamfer_grid_bytes(n1, n2));
        double *cd = filled<double>(8);
        float *grad2 = filled<float>(12ull * n2);
        int32_t *nn12 = filled<int32_t>(4ull * n1), *nn21 = filled<int32_t>(4ull * n2);
        if (dpr::launch_chamfer_grid(n1, s1, n2, s2, cd, grad2, nn12, nn21, ws, nullptr) != hipSuccess) return 3;
        write_raw(dir + "/cd.bin", cd, 8);
        write_raw(dir + "/grad2.bin", grad2, 12ull * n2);
        write_raw(dir + "/nn12.bin", nn12, 4ull * n1);
        write_raw(dir + "/nn21.bin", nn21, 4ull * n2);
        std::free(ws); std::free(cd); std::free(grad2); std::free(nn12); std::free(nn21);
    } else if (mode == "topk" && argc == 5) {
        const int k3 = std::atoi(argv[3]), K = std::atoi(argv[4]);
        float *sh1 = read_f32(dir + "/sh1.bin", &fh);
        uint8_t *ws = filled<uint8_t>(dpr::topk_grid_bytes(n1, n2, K));
        float *out = filled<float>(4ull * n2 * (uint64_t)k3);
        int32_t *idx = filled<int32_t>(4ull * n2 * (uint64_t)K);
        if (dpr::launch_topk_grid(n1, s1, sh1, n2, s2, k3, K, out, idx, ws, nullptr) != hipSuccess) return 3;
        write_raw(dir + "/out_sh.bin", out, 4ull * n2 * (uint64_t)k3);
        write_raw(dir + "/idx.bin", idx, 4ull * n2 * (uint64_t)K);
        std::free(ws); std::free(sh1); std::free(out); std::free(idx);
    } else {
        return 2;
    }
    std::free(s1);
    std::free(s2);
    return 0;
}
