// Mesh passes of the axis lengths of group b (mesh_len.h).
#include "mesh_len_launch.h"

#define LENGTHS(X) X(12) X(64) X(108) X(200) X(500)
QEQ_LEN_GROUP(mesh_len_b, LENGTHS)
