// Bytes from a control block's stored tolerance to its two counts.
#include <cstdio>

#include "ff_internal.h"

int main() {
    const size_t tol = offsetof(ff::Ctl, p) + offsetof(ff::MinParamsDev, tol);
    std::printf("%zu %zu\n", offsetof(ff::Ctl, fin_ticket) - tol, offsetof(ff::Ctl, acc_ticket) - tol);
}
