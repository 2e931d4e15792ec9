// A HIP runtime on the host for tests of the library's host code: device memory
// is host memory, copies and fills are done, launches are recorded and do
// nothing.  (tests/_hostcode.py links it in the runtime's place.)
#pragma once
#include <hip/hip_runtime.h>

#include <string>
#include <vector>

namespace fake {

struct Launch {
    std::string kernel;   // as declared, with its template arguments
    dim3 grid, block;
    size_t lds;           // dynamic
    int device;
};
struct Limit {            // hipFuncSetAttribute (dynamic LDS)
    std::string kernel;
    int bytes, device;
};
extern std::vector<Launch> launches;
extern std::vector<Limit> limits;
extern std::vector<size_t> mallocs;
extern int device;        // the current one
std::vector<std::string> kernels();   // every kernel that the library holds

inline bool has(const std::string &s, const char *part) { return s.find(part) != std::string::npos; }

}  // namespace fake
