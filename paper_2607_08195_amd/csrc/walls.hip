// The parked particles of a step: re-emission at diffuse walls and the rest of
// their flight.  A file of its own, compiled without the hoisting of constants
// out of loops (the coefficients of FP64 sine, cosine and logarithm would take
// a wave per SIMD of this kernel, while the move kernel fares better with it).
#include "kernels.h"

namespace dsmcx {

// Finishes the step of the parked particles, one queue entry per lane at a
// time: a particle parked at a diffuse wall is re-emitted there, one parked in
// flight resumes with its velocity; walls reached later are re-emitted from by
// the same code at the head of the loop (a copy of it in the hop loop cost 40
// registers, a wave per SIMD).  Workgroups take the queue parts round-robin
// (gridDim.x is a multiple of kQueueParts) and stride through their part.
// (Refilling lanes from the queue as their particles finish was measured
// slower: the refill brings the scattered loads and the wall re-emission into
// every pass of the hop loop.)  Bound by the latency of the longest tracks.
// SURF = false: surface sampling is off.  127 us for the 2.76M particles of a
// batch of cavities (145 with 161 registers instead of 128), 77 on the 40^3
// cavity, 35 for 26,000 particles at Kn 1.
template <class VT, bool SURF>
__global__ __launch_bounds__(256) void k_move_walls(MeshDev m, PartDev<VT> p, const Scalars* sc, int32_t* counts,
                                                   uint32_t* rank, Counters* ctr, RngKey key, WallQueue q) {
    const int part = (int)(blockIdx.x % kQueueParts);
    const int64_t nq = (int64_t)q.n[(size_t)part * kQueueStride];
    const int64_t stride = (int64_t)(gridDim.x / kQueueParts) * blockDim.x;
    const uint32_t step = sc->step;
    int hops = 0, walls = 0, rem = 0, lost = 0;
    for (int64_t k = (int64_t)(blockIdx.x / kQueueParts) * blockDim.x + threadIdx.x; k < nq; k += stride) {
        const int64_t e = part * q.part + k;
        const int64_t i = q.idx[e];
        const int meta = q.meta[e];
        const double tq = q.t[e];
        Walker w;
        w.x0 = p.pos[3 * i]; w.x1 = p.pos[3 * i + 1]; w.x2 = p.pos[3 * i + 2];
        w.c = p.cell[i]; w.pid = p.pid[i]; w.t = tq < 0 ? -tq : tq;
        w.entry = meta & 3; w.hits = (meta >> 2) & 1023; w.nhop = (meta >> 12) & 1023; w.walls = (meta >> 22) & 1023;
        if (m.rot) w.ir = p.ir[i];
        RngKey kp = key;
        double dtp = 0.0;
        case_params(m.cell_case, m.cases, w.c, kp, dtp);
        // a walker parked in flight carries a negative time; one parked at a
        // diffuse wall entered through a boundary face.  Both tests are made:
        // a non-finite time (a particle whose position lies in no cell) has no
        // usable sign, and only a boundary face may be re-emitted from.
        int code = m.nbr[4 * w.c + w.entry];
        bool pend = !(tq < 0 || code >= 0);
        // (surface sampling needs the velocity the particle reached the wall with)
        if (SURF || !pend) {
            w.v0 = (double)p.vel[3 * i]; w.v1 = (double)p.vel[3 * i + 1]; w.v2 = (double)p.vel[3 * i + 2];
        }
        int st;
        do {
            if (pend) diffuse_reemit<VT, SURF>(m, w, -1 - code, w.entry, step, kp);
            st = hop_once<VT, true, true, SURF>(m, w, step, kp);  // parked walkers have an entry face
            pend = st == kHopWallPending;
            if (pend) code = m.nbr[4 * w.c + w.entry];
        } while (st < 0 || pend);
        hops += w.nhop;
        walls += w.walls;
        p.pos[3 * i] = w.x0; p.pos[3 * i + 1] = w.x1; p.pos[3 * i + 2] = w.x2;
        p.vel[3 * i] = (VT)w.v0; p.vel[3 * i + 1] = (VT)w.v1; p.vel[3 * i + 2] = (VT)w.v2;
        if (m.rot) p.ir[i] = w.ir;
        if (st == 0) {
            p.cell[i] = w.c;
            rank[i] = (uint32_t)atomicAdd(&counts[w.c], 1);
        } else {
            p.cell[i] = -1;
            rem += st == 1;
            lost += st == 2;
        }
    }
    block_counters(hops, walls, rem, lost, &ctr->hops, &ctr->walls, &ctr->removed, &ctr->lost);
}

template <class VT>
void launch_move_walls(hipStream_t s, const MeshDev& m, PartDev<VT> p, const Scalars* sc, int32_t* counts,
                       uint32_t* rank, Counters* ctr, RngKey key, WallQueue wq) {
    const auto k = m.surf ? k_move_walls<VT, true> : k_move_walls<VT, false>;
    hipLaunchKernelGGL(k, dim3(1024), dim3(256), 0, s, m, p, sc, counts, rank, ctr, key, wq);
}

template void launch_move_walls<float>(hipStream_t, const MeshDev&, PartDev<float>, const Scalars*, int32_t*, uint32_t*,
                                       Counters*, RngKey, WallQueue);
template void launch_move_walls<double>(hipStream_t, const MeshDev&, PartDev<double>, const Scalars*, int32_t*,
                                        uint32_t*, Counters*, RngKey, WallQueue);

}  // namespace dsmcx
