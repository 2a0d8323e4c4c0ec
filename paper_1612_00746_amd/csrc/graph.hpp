// One particle on a general graph (see graph.hip).
#pragma once
#include "ctqw_internal.hpp"

namespace ctqw {

// One Taylor term of every realisation: t = (-i c) H src, acc_out = acc_in + t.
// Pointers are untyped: complex64 states with FP32 tables, or complex128
// states with FP64 tables (dtype 0 / 1).
struct GraphTermArgs {
    const int32_t* nbr;      // [width][n] neighbour of node i in slot k; outside [0, n): empty slot
    const void* hop;         // [R][width][n] coupling of that slot
    const void* onsite;      // [R][n] diagonal
    const void* src;         // [R][n] the previous term (or the state)
    void* t_out;             // [R][n] this term, or NULL when no later term needs it
    const void* acc_in;      // [R][n] partial sum before this term
    void* acc_out;           // [R][n] partial sum after it, or NULL: the next term adds this one
    double* parts;           // [R][ceil(n / 256)] parts of acc_out's squared norms, or NULL
    int32_t add_src;         // the sum takes the source first (the term that left it out)
    double c;                // dt / j for term j
    int32_t n;
    int32_t width;
    int32_t R;
    int32_t node_blocks;     // set by the launcher
    int32_t by_xcd;
};
hipError_t launch_graph_term(const GraphTermArgs& a, int dtype, hipStream_t s);
// out[r] = the sum of the parts of realisation r, in a fixed order.
hipError_t launch_graph_norms(const double* parts, int32_t n, int32_t R, double* out, hipStream_t s);

}  // namespace ctqw
