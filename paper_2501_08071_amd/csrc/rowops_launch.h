// Internal: host-side launch interface of the row kernels (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>

struct RowopLaunch {
    int op;            // 0 softmax, 1 rmsnorm
    const void* x;
    const void* w;     // rmsnorm only
    void* y;
    long long n_rows;
    int n;             // row length
    float eps;
    int dtype;         // 0 binary16, 1 bfloat16
    void* stream;
};

constexpr int ROWOPS_MAX_REG_ROW = 65536;   // longest row kept in registers between its read and its write (1024 threads x 8 chunks x 8)

// 1 = rows of up to 16384 elements that start at 16-byte aligned addresses, 2 = other lengths
inline int rowop_path_of(int n) { return (n % 8 == 0 && n <= 16384) ? 1 : 2; }

hipError_t rowop_launch(const RowopLaunch& a);
