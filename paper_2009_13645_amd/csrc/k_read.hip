// k_read.hip -- read-back kernels: one field component or the particle state
// laid out on the device as the caller's host array is, so that a read call
// is one kernel and plain copies.
//
// What bounds them: the copy to the host (D2H), tens of GB/s against
// terabytes per second on the device.  So each kernel moves as few bytes
// over to the host as the call returns and does the reordering and the
// type conversion here.  Before, E and B were read by evaluating all six
// components into the interleaved vertex array and copying all eight words
// of every node (96 x 96 x 256 nodes at FP32: 19.5 ms a component, now 0.58),
// and the particles by column copies and a scatter by id on the host
// (1.5 million: 27 ms, now 7.9).
#include "mithra_dev.hpp"

namespace mithra {

// out[n] = a[n] (+ lo[n]), in the caller's type
template <typename T, typename O>
__global__ __launch_bounds__(256) void k_read_convert(const T *a, const T *lo, O *out, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        out[i] = (O)((double)a[i] + (lo ? (double)lo[i] : 0.0));
}

// Component `id` (0..2: E, 3..5: B) at every node from the potentials of step
// s, zero on the boundary: the vertex formulas of the step (VertexFields),
// rounded to the run's field type as the step's are.  One thread per node,
// x fastest; a wavefront's neighbour reads hit the lines its own nodes use.
template <typename T, typename O>
__global__ __launch_bounds__(256) void k_read_vertex(RunDev R, int64_t s, int id, O *out)
{
    const int a = id < 3 ? id : id - 3, m1 = a == 2 ? 0 : a + 1, m2 = a == 0 ? 2 : a - 1;
    const T *An = pot_ptr<T>(R, slot_cur(s), a), *Ap = pot_ptr<T>(R, slot_next(s), a);
    const T *An1 = pot_ptr<T>(R, slot_cur(s), m1), *Ap1 = pot_ptr<T>(R, slot_next(s), m1);
    const T *An2 = pot_ptr<T>(R, slot_cur(s), m2), *Ap2 = pot_ptr<T>(R, slot_next(s), m2);
    const T *ph = pot_ptr<T>(R, slot_cur(s), 3);
    auto stride = [&](int ax) { return ax == 0 ? (int64_t)1 : (ax == 1 ? (int64_t)R.nx : (int64_t)R.nx * R.ny); };
    auto half = [&](int ax) { return 0.5 / (ax == 0 ? R.dx : (ax == 1 ? R.dy : R.dz)); };
    const int64_t sa = stride(a), s1 = stride(m1), s2 = stride(m2);
    const double ia = half(a), i1 = half(m1), i3 = half(m2);
    const uint32_t nx = (uint32_t)R.nx, ny = (uint32_t)R.ny;  // nodes <= 4e9: 32-bit decoding
    for (int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x; c < R.nn; c += (int64_t)gridDim.x * 256) {
        const uint32_t row = (uint32_t)c / nx, k = row / ny;
        const int i = (int)((uint32_t)c - row * nx), j = (int)(row - k * ny);
        double v = 0.0;
        if (i > 0 && i < R.nx - 1 && j > 0 && j < R.ny - 1 && k > 0 && (int)k < R.nz - 1) {
            auto dif = [c](const T *f, int64_t d) { return (double)f[c + d] - (double)f[c - d]; };
            if (id < 3) {
                const double g = R.space_charge ? dif(ph, sa) * ia : 0.0;
                v = -((double)Ap[c] - (double)An[c]) / R.dt - g;
            } else {
                v = 0.5 * ((dif(An2, s1) + dif(Ap2, s1)) * i1 - (dif(An1, s2) + dif(Ap1, s2)) * i3);
            }
        }
        out[c] = (O)(T)v;
    }
}

// Particles in id order: xyz and u as rows of three, the linear cell index
// (-1 outside the active region) and the ids in the current sort order (the
// slots of the last sort, or the buffer order when no sort followed the last
// push).  Any output may be null.
__global__ __launch_bounds__(256) void k_read_particles(RunDev R, double *xyz, double *u, int32_t *cell, int32_t *order)
{
    const int pb = R.ctl->pbuf, sb = R.ctl->sorted_buf;
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= R.np)
        return;
    const int64_t id = R.pid[pb][p];
    const double r[3] = {R.pr[pb][0][p], R.pr[pb][1][p], R.pr[pb][2][p]};
    if (xyz)
        for (int a = 0; a < 3; ++a)
            xyz[3 * id + a] = r[a];
    if (u)
        for (int a = 0; a < 3; ++a)
            u[3 * id + a] = R.pr[pb][3 + a][p];
    if (cell) {
        const double g[3] = {(r[0] - R.x0) / R.dx, (r[1] - R.y0) / R.dy, (r[2] - R.z0) / R.dz};
        const int n[3] = {R.nx, R.ny, R.nz};
        int c[3];
        bool act = true;
        for (int a = 0; a < 3; ++a) {
            const double f = floor(g[a]);
            act = act && f >= 1.0 && f <= (double)(n[a] - 3);
            c[a] = act ? (int)f : 0;
        }
        cell[id] = act ? (int32_t)nid(R, c[0], c[1], c[2]) : -1;
    }
    if (order)
        order[p] = R.pid[pb][sb < 0 ? p : (int64_t)R.sv[sb][p]];
}

// The field array `a` (plus its compensation terms `lo`, or null) of the
// run's type as FP64 (out64) or FP32.
hipError_t launch_read_convert(const RunDev &R, const void *a, const void *lo, void *out, bool out64, hipStream_t st)
{
    const int64_t b = (R.nn + 255) / 256;
    const dim3 g((unsigned)(b > 16384 ? 16384 : b));
    if (R.precision == 32 && out64)
        hipLaunchKernelGGL((k_read_convert<float, double>), g, dim3(256), 0, st, (const float *)a, (const float *)lo,
                           (double *)out, R.nn);
    else if (R.precision == 32)
        hipLaunchKernelGGL((k_read_convert<float, float>), g, dim3(256), 0, st, (const float *)a, (const float *)lo,
                           (float *)out, R.nn);
    else
        hipLaunchKernelGGL((k_read_convert<double, float>), g, dim3(256), 0, st, (const double *)a, (const double *)lo,
                           (float *)out, R.nn);
    return hipGetLastError();
}

hipError_t launch_read_vertex(const RunDev &R, int64_t s, int id, void *out, bool out64, hipStream_t st)
{
    const int64_t b = (R.nn + 255) / 256;
    const dim3 g((unsigned)(b > 16384 ? 16384 : b));
    if (R.precision == 32 && out64)
        hipLaunchKernelGGL((k_read_vertex<float, double>), g, dim3(256), 0, st, R, s, id, (double *)out);
    else if (R.precision == 32)
        hipLaunchKernelGGL((k_read_vertex<float, float>), g, dim3(256), 0, st, R, s, id, (float *)out);
    else if (out64)
        hipLaunchKernelGGL((k_read_vertex<double, double>), g, dim3(256), 0, st, R, s, id, (double *)out);
    else
        hipLaunchKernelGGL((k_read_vertex<double, float>), g, dim3(256), 0, st, R, s, id, (float *)out);
    return hipGetLastError();
}

hipError_t launch_read_particles(const RunDev &R, double *xyz, double *u, int32_t *cell, int32_t *order,
                                 hipStream_t st)
{
    hipLaunchKernelGGL(k_read_particles, dim3((unsigned)((R.np + 255) / 256)), dim3(256), 0, st, R, xyz, u, cell,
                       order);
    return hipGetLastError();
}

}  // namespace mithra
