// Mesh passes of the axis lengths of group h (mesh_len.h).
#include "mesh_len_launch.h"

#define LENGTHS(X) X(32) X(180) X(320) X(324)
QEQ_LEN_GROUP(mesh_len_h, LENGTHS)
