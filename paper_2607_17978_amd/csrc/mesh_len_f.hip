// Mesh passes of the axis lengths of group f (mesh_len.h).
#include "mesh_len_launch.h"

#define LENGTHS(X) X(72) X(100) X(288) X(384)
QEQ_LEN_GROUP(mesh_len_f, LENGTHS)
